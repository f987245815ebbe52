// robustPrune (Alg. 3) for uint8 vectors of at most 256 bytes: one wavefront per prune, 32 pivots per round.
//
// The candidates are in (distance, id) order.  A round takes the next 32 live ones as pivots and holds their vectors as
// MFMA operands.  One 32 x 32 tile gives the relation among the pivots, from which a fixpoint on bit masks decides which
// of them Alg. 3 selects (a pivot with a selected discarder is dead, one whose discarders are all dead is selected; the
// first undecided one is always decided, so it ends).  The live candidates behind them follow in blocks of 32, the next
// block's vectors on their way while one is tested: a tile against the pivots, the bits of the selected ones, and the
// survivors are written back to the list, still in order.  So a round costs one memory latency, and what an early
// selection discards (most of a list) is never looked at again.
//
// A test is alpha * d(i,j) <= d(p,j) in float32, d(i,j) = |x_i|^2 + |x_j|^2 - 2 <x_i, x_j> from v_mfma_i32_32x32x32_i8 on
// the values shifted by -128, exact.  Distances are below 2^24, so they convert to float32 exactly, and a float32 product
// by alpha does not decrease with d: "i discards j" is d(i,j) <= t_j with the largest integer t_j for which it holds,
// found once per candidate, and three vector instructions per pair: 2 <x_i, x_j> - |x_i|^2 >= |x_j|^2 - t_j, and the bit
// shifted into a mask.
//
// What bounds it: vector instructions (about 120 for a block against 32 pivots), and with few prunes the four to six rounds
// of a list, a memory latency each.  Forward prune of 37,500 expansion lists (about 190 entries) 519 -> 142 us, of 32 43 -> 9
// (before: four pivots per round on dot products); the reverse merges of a build of 200,000 x 128 12.2 -> 2.6 ms (a list or
// a 128-slot Gram matrix per wavefront, rows that remembered their last prune, hubs in one wavefront's selection loop); the
// prunes of a consolidation of 180,000 rows 7.3 -> 1.1 ms.  A build of 100,000 x 256 37.8 -> 16.5 ms.
#include "jx_distance.h"

namespace jx {

typedef int gi32x16_t __attribute__((ext_vector_type(16)));
typedef int gi32x4_t __attribute__((ext_vector_type(4)));

template <int MAXC>
struct PivotLds {
    uint32_t id[MAXC];
    float dx[MAXC];        // d(p, candidate)
    int kk[MAXC];          // |x_j|^2 - t_j
    uint16_t list[MAXC];   // live candidates, in order
    int pn[32];            // -|x|^2 of the pivots, by operand row
    uint16_t kw[64];       // relation among the pivots: [pivot][half], bit = a pivot that discards it
    // a row's present neighbours while a list is put together: keys as read and in order, new edges right before each
    uint64_t fixed[JX_MAX_R];
    union {
        uint64_t raw[JX_MAX_R];
        struct {
            uint32_t sel_id[JX_MAX_R];
            uint32_t sel_dist[JX_MAX_R];
        };
    };
    uint32_t count[JX_MAX_R];
};

// Operand of a lane: 16 bytes of row lane % 32 for each of 4 S steps, chunk 2 step + lane / 32
template <int S>
struct Frag {
    uint4 x[4 * S];
    __device__ __forceinline__ void load(const uint8_t* rec, int half, int nch) {
        if (nch == 8 * S) {  // uniform
#pragma unroll
            for (int k = 0; k < 4 * S; k++) x[k] = load16(rec + (2 * k + half) * 16);
        } else {
#pragma unroll
            for (int k = 0; k < 4 * S; k++) {
                const int ch = 2 * k + half;
                x[k] = load16(rec + (ch < nch ? ch : 0) * 16);
                if (ch >= nch) x[k] = make_uint4(0x80808080u, 0x80808080u, 0x80808080u, 0x80808080u);  // zero after the shift
            }
        }
    }
    __device__ __forceinline__ void shift() {
#pragma unroll
        for (int k = 0; k < 4 * S; k++) {
            x[k].x ^= 0x80808080u;
            x[k].y ^= 0x80808080u;
            x[k].z ^= 0x80808080u;
            x[k].w ^= 0x80808080u;
        }
    }
};

// sum over both lanes of a row
template <int S>
__device__ __forceinline__ int frag_dot(const Frag<S>& a, const Frag<S>& b) {
    int t = 0;
#pragma unroll
    for (int k = 0; k < 4 * S; k++) {
        t = __builtin_amdgcn_sdot4((int)a.x[k].x, (int)b.x[k].x, t, false);
        t = __builtin_amdgcn_sdot4((int)a.x[k].y, (int)b.x[k].y, t, false);
        t = __builtin_amdgcn_sdot4((int)a.x[k].z, (int)b.x[k].z, t, false);
        t = __builtin_amdgcn_sdot4((int)a.x[k].w, (int)b.x[k].w, t, false);
    }
    return t + shfl_xor(t, 32);
}

// largest integer t with (float)alpha * (float)t <= d, or -1
__device__ __forceinline__ int discard_limit(float d, float alpha) {
    int t = (int)(d / alpha);  // off by one or two at most: quotient and products are below 2^24
#pragma unroll
    for (int s = 0; s < 3; s++)
        if (t >= 0 && !(__fmul_rn(alpha, (float)t) <= d)) t--;
#pragma unroll
    for (int s = 0; s < 3; s++)
        if (t >= 0 && __fmul_rn(alpha, (float)(t + 1)) <= d) t++;
    return t;
}

// bits e = 0..15: pivot of accumulator row e discards the lane's column
template <int S>
__device__ __forceinline__ uint32_t discard_bits(const Frag<S>& a, const Frag<S>& b, const int (&negn)[16], int kj) {
    gi32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0;
#pragma unroll
    for (int k = 0; k < 4 * S; k++)
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(gi32x4_t, a.x[k]), __builtin_bit_cast(gi32x4_t, b.x[k]), acc, 0, 0, 0);
    uint32_t w = 0;
#pragma unroll
    for (int e = 15; e >= 0; e--) w = w + w + ((acc[e] << 1) + negn[e] >= kj ? 1u : 0u);
    return w;
}

// L->id / L->dx [0..m) in (distance, id) order.  Returns the number selected (at most R), L->sel_id / L->sel_dist.
template <int S, int MAXC>
__device__ __forceinline__ int pivot_prune(PivotLds<MAXC>* L, const uint8_t* recs, size_t stride, int nch, int m, uint32_t p, int R,
                                           float alpha) {
    const int lane = lane_id(), col = lane & 31, half = lane >> 5;
    // accumulator register e of half h is row 8 (e / 4) + 4 h + e % 4: bit e + 16 h of a mask.  Operand row `col` holds
    // the pivot of that number, so that masks are in the order of the pivots
    const int q = (((col >> 3) << 2) | (col & 3)) + 16 * ((col >> 2) & 1);
    int n = 0;
    for (int j0 = 0; j0 < m; j0 += 64) {
        const int j = j0 + lane;
        const bool on = j < m && L->id[j < m ? j : 0] != p;
        const uint64_t b = ballot(on);
        if (on) L->list[n + prefix_count(b)] = (uint16_t)j;
        n += __builtin_popcountll(b);
    }
    wave_sync();
    int nsel = 0;
    bool first = true;
    while (n > 0 && nsel < R) {
        const int np = n < 32 ? n : 32;
        const int slot = L->list[q < np ? q : 0];
        Frag<S> a, b;
        a.load(recs + (size_t)L->id[slot] * stride, half, nch);
        int vs = 0;
        if (n > 32) {
            vs = L->list[32 + col < n ? 32 + col : n - 1];
            b.load(recs + (size_t)L->id[vs] * stride, half, nch);
        }
        a.shift();
        const int na = frag_dot(a, a);
        int kj;
        if (first) {
            kj = na - discard_limit(L->dx[slot], alpha);
            if (half == 0) L->kk[slot] = kj;
        } else {
            kj = L->kk[slot];
        }
        if (half == 0) L->pn[col] = -na;
        wave_sync();
        int negn[16];
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const int4 x = *reinterpret_cast<const int4*>(&L->pn[8 * g + 4 * half]);
            negn[4 * g] = x.x;
            negn[4 * g + 1] = x.y;
            negn[4 * g + 2] = x.z;
            negn[4 * g + 3] = x.w;
        }
        L->kw[2 * q + half] = (uint16_t)discard_bits<S>(a, a, negn, kj);
        wave_sync();
        const uint32_t before = (1u << col) - 1u;
        const uint32_t w = reinterpret_cast<const uint32_t*>(L->kw)[col] & before;
        uint32_t U = np == 32 ? 0xFFFFFFFFu : (1u << np) - 1u, sel = 0;
        while (U) {
            const uint32_t dead = (uint32_t)ballot((w & sel) != 0) & U;
            const uint32_t take = (uint32_t)ballot((w & (sel | U)) == 0) & U;
            U &= ~(dead | take);
            sel |= take;
        }
        if (half == 0 && ((sel >> col) & 1u)) {
            const int pos = nsel + __builtin_popcount(sel & before);
            if (pos < R) {
                const int s = L->list[col];
                L->sel_id[pos] = L->id[s];
                L->sel_dist[pos] = __float_as_uint(L->dx[s]);
            }
        }
        nsel += __builtin_popcount(sel);
        const uint32_t mine = half ? sel >> 16 : sel & 0xFFFFu;
        int left = 0;
        for (int v0 = 32; v0 < n && nsel < R; v0 += 32) {
            Frag<S> nx;
            int ns = 0;
            if (v0 + 32 < n) {
                ns = L->list[v0 + 32 + col < n ? v0 + 32 + col : n - 1];
                nx.load(recs + (size_t)L->id[ns] * stride, half, nch);
            }
            b.shift();
            int kv;
            if (first) {
                kv = frag_dot(b, b) - discard_limit(L->dx[vs], alpha);
                if (half == 0) L->kk[vs] = kv;
            } else {
                kv = L->kk[vs];
            }
            const uint64_t dead = ballot((discard_bits<S>(a, b, negn, kv) & mine) != 0);
            const int in = n - v0;
            const uint32_t live = ~((uint32_t)dead | (uint32_t)(dead >> 32)) & (in >= 32 ? 0xFFFFFFFFu : (1u << in) - 1u);
            // in place: survivors move down, behind what is read next
            if (half == 0 && ((live >> col) & 1u)) L->list[left + __builtin_popcount(live & before)] = (uint16_t)vs;
            left += __builtin_popcount(live);
            b = nx;
            vs = ns;
        }
        n = left;
        first = false;
        wave_sync();
    }
    return nsel < R ? nsel : R;
}

// ---- forward prune of the candidate list of each new point (Alg. 4 step 2)
template <int S, int MAXC>
__global__ void __launch_bounds__(64) forward_prune_u8_kernel(InsertArgs a) {
    __shared__ PivotLds<MAXC> lds;
    PivotLds<MAXC>* L = &lds;
    const int lane = lane_id();
    const long long i = blockIdx.x;
    long long xid = a.id_base + i;
    if (xid >= a.id_skip) xid++;
    const uint32_t* ids = a.cand_ids + (size_t)i * a.L;
    const uint32_t* dbits = a.cand_dist + (size_t)i * a.L;
    int m = 0;
#pragma unroll
    for (int h = 0; h < MAXC / 64; h++) {
        const int j = h * 64 + lane;
        uint32_t id = JX_NONE_ID;
        if (j < a.L) id = ids[j];
        if (id != JX_NONE_ID) {
            L->id[j] = id;
            L->dx[j] = __uint_as_float(dbits[j]);
        }
        m += __builtin_popcountll(ballot(id != JX_NONE_ID));  // the list is filled from the left
    }
    wave_sync();
    const int nsel = pivot_prune<S, MAXC>(L, a.ds.recs, (size_t)a.ds.rec_stride, a.ds.nch, m, (uint32_t)xid, a.R, a.alpha);
    wave_sync();
    if (lane == 0) a.clean[xid] = (uint8_t)(nsel < 255 ? nsel : 255);
    uint32_t* row = a.adj + (size_t)xid * a.R;
    for (int j = lane; j < a.R; j += 64) {
        const bool on = j < nsel;
        const uint32_t v = on ? L->sel_id[j] : JX_NONE_ID;
        row[j] = v;
        a.keys[(size_t)i * a.R + j] = on ? (((uint64_t)v << 32) | L->sel_dist[j]) : JX_EMPTY_KEY;
        a.vals[(size_t)i * a.R + j] = on ? (uint32_t)xid : JX_NONE_ID;
    }
}

// ---- reverse-edge merge of a row whose first c entries one robustPrune selected together (they stand in (distance, id) order and
// none discards another), with k - 1 <= 15 appended entries and new edges behind them: the fresh ones.  Only pairs with a fresh
// one have to be tested.  In order of distance a fresh entry is dead if one that is alive and comes before it discards it; else it
// stays, and what it discards is dead from then on.  p and the fresh vectors are the rows of a tile, the clean ones the
// columns of one or two, so every vector is read once and the chain has one memory latency, where rounds of pivots have
// one for the distances and one for each round.  Full rows that get an edge now and then, which is what a stream into a large
// index consists of, take this way: 100,000 points into 8M 20.8 -> 17.3 ms, into 20M 29.4 -> 23.1 (26.7 by the list-based kernel
// of few fresh entries that stood here before the rounds of pivots).
template <int S>
__device__ __forceinline__ int merge_fresh(const InsertArgs& a, const uint32_t v, uint32_t* row, const int c, const int deg, const int k,
                                           const long long lo) {
    const int lane = lane_id(), col = lane & 31, half = lane >> 5;
    const size_t stride = (size_t)a.ds.rec_stride;
    uint32_t iid = v;  // items: 0 = v, 1 .. k = the fresh ones
    if (col >= 1 && col <= k) {
        const int f = col - 1;
        iid = f < deg - c ? row[c + f] : a.vals[lo + f - (deg - c)];
    }
    uint32_t cid[2];
#pragma unroll
    for (int b = 0; b < 2; b++) cid[b] = row[b * 32 + col < c ? b * 32 + col : 0];
    const int nb = c > 32 ? 2 : 1;  // uniform
    Frag<S> it, x[2];
    it.load(a.ds.recs + (size_t)iid * stride, half, a.ds.nch);
    x[0].load(a.ds.recs + (size_t)cid[0] * stride, half, a.ds.nch);
    if (nb == 2) x[1].load(a.ds.recs + (size_t)cid[1] * stride, half, a.ds.nch);
    it.shift();
    const int ni = frag_dot(it, it), np = (int)readlane32((uint32_t)ni, 0);
    uint32_t dis[3] = {}, vic[3] = {};  // lane r, item r: what discards it and what it discards among the clean ones 0 .. 31, 32 .. 63, the items
    uint64_t kx[3];                     // (distance, id) of the lane's column
    // the tile of one set of columns
    auto tile = [&](const Frag<S>& y, const int ny, const uint32_t id, const bool on, const int b) __attribute__((always_inline)) {
        gi32x16_t acc;
#pragma unroll
        for (int e = 0; e < 16; e++) acc[e] = 0;
#pragma unroll
        for (int s = 0; s < 4 * S; s++)
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(gi32x4_t, it.x[s]), __builtin_bit_cast(gi32x4_t, y.x[s]), acc, 0, 0, 0);
        const int other = shfl_xor(acc[0], 32), dp = half ? other : acc[0];  // row 0 is with the first half
        const float dx = (float)(uint32_t)(np + ny - 2 * dp);
        kx[b] = ((uint64_t)__float_as_uint(dx) << 32) | id;
#pragma unroll
        for (int e = 0; e < 8; e++) {  // rows r0 and r0 + 4: accumulator register e of half h is row 8 (e / 4) + 4 h + e % 4
            const int r0 = 8 * (e >> 2) + (e & 3), r = r0 + 4 * half;
            if (r0 > k) continue;  // uniform
            const uint64_t kf0 = readlane64(kx[2], r0), kf1 = readlane64(kx[2], r0 + 4), kf = half ? kf1 : kf0;
            const int nf0 = (int)readlane32((uint32_t)ni, r0), nf1 = (int)readlane32((uint32_t)ni, r0 + 4);
            const float ad = __fmul_rn(a.alpha, (float)(uint32_t)(ny + (half ? nf1 : nf0) - 2 * acc[e]));
            const bool pair = on && r >= 1 && r <= k;
            const uint64_t out = ballot(pair && kf < kx[b] && ad <= dx);
            const uint64_t in = ballot(pair && kx[b] < kf && ad <= __uint_as_float((uint32_t)(kf >> 32)));
            if (lane == r0) {
                vic[b] = (uint32_t)out;
                dis[b] = (uint32_t)in;
            }
            if (lane == r0 + 4) {
                vic[b] = (uint32_t)(out >> 32);
                dis[b] = (uint32_t)(in >> 32);
            }
        }
    };
    tile(it, ni, iid, col >= 1 && col <= k, 2);  // first: the fresh ones' own distances
    kx[1] = JX_EMPTY_KEY;
    x[0].shift();
    tile(x[0], frag_dot(x[0], x[0]), cid[0], col < c, 0);
    if (nb == 2) {
        x[1].shift();
        tile(x[1], frag_dot(x[1], x[1]), cid[1], 32 + col < c, 1);
    }
    // ---- Alg. 3
    uint32_t alive0 = c >= 32 ? 0xFFFFFFFFu : (1u << c) - 1u, alive1 = c >= 64 ? 0xFFFFFFFFu : (c > 32 ? (1u << (c - 32)) - 1u : 0u), alivef = 0;
    int place = 0;
    for (int t = 1; t <= k; t++) place += readlane64(kx[2], t) < kx[2] ? 1 : 0;
    for (int s = 0; s < k; s++) {
        uint32_t next = (uint32_t)ballot(lane >= 1 && lane <= k && place == s);
        for (; next; next &= next - 1u) {
            const int r = __builtin_ctz(next);
            if ((readlane32(dis[0], r) & alive0) | (readlane32(dis[1], r) & alive1) | (readlane32(dis[2], r) & alivef)) continue;
            alive0 &= ~readlane32(vic[0], r);
            alive1 &= ~readlane32(vic[1], r);
            alivef |= 1u << r;
        }
    }
    int nsel = c;
    if (alivef) {  // else the clean ones stay where they are
        const uint32_t before = (1u << col) - 1u;
        int at0 = __builtin_popcount(alive0 & before), at1 = __builtin_popcount(alive0) + __builtin_popcount(alive1 & before), atf = 0;
        for (uint32_t w = alivef; w; w &= w - 1u) {
            const int f = __builtin_ctz(w);
            const uint64_t kf = readlane64(kx[2], f);
            const int ahead = __builtin_popcount(alive0 & ~(uint32_t)ballot(kf < kx[0])) + __builtin_popcount(alive1 & ~(uint32_t)ballot(kf < kx[1]));
            at0 += kf < kx[0] ? 1 : 0;
            at1 += kf < kx[1] ? 1 : 0;
            atf += (kf < kx[2] ? 1 : 0) + (lane == f ? ahead : 0);
        }
        if (half == 0 && ((alive0 >> col) & 1u) && at0 != col && at0 < a.R) row[at0] = cid[0];
        if (half == 1 && ((alive1 >> col) & 1u) && at1 != 32 + col && at1 < a.R) row[at1] = cid[1];
        if (half == 0 && ((alivef >> col) & 1u) && atf < a.R) row[atf] = iid;
        nsel = __builtin_popcount(alive0) + __builtin_popcount(alive1) + __builtin_popcount(alivef);
        if (nsel > a.R) nsel = a.R;
    }
    for (int j = nsel + lane; j < deg; j += 64) row[j] = JX_NONE_ID;
    return nsel;
}

// The segments that reverse_class_kernel has listed for it
template <int S>
__global__ void __launch_bounds__(64, S == 1 ? 4 : 1) reverse_merge_fresh_u8_kernel(InsertArgs a) {
    const int lane = lane_id();
    const uint32_t n = a.nseg[3];
    const long long total = a.B * a.R;
    for (uint32_t at = blockIdx.x; at < n; at += gridDim.x) {
        const uint32_t s = a.fresh[at], lo = a.heads[s];
        const uint32_t v = (uint32_t)(a.keys[lo] >> 32);
        const uint32_t* keys_hi = reinterpret_cast<const uint32_t*>(a.keys) + 1;
        const int m = __builtin_popcountll(ballot(lane < 16 && lo + lane < total && keys_hi[2 * (size_t)(lo + (lane < 16 ? lane : 0))] == v));
        uint32_t* row = a.adj + (size_t)v * a.R;
        const int c = a.clean[v];
        int deg = 0;
        for (int r = 0; r < a.R; r += 64) deg += __builtin_popcountll(ballot(r + lane < a.R && row[r + lane] != JX_NONE_ID));
        const int nsel = merge_fresh<S>(a, v, row, c, deg, deg - c + m, lo);
        if (lane == 0) {
            a.clean[v] = (uint8_t)nsel;
            const_cast<uint32_t*>(a.heads)[s] = lo | 0x80000000u;
        }
    }
}

// ---- reverse-edge merge (Alg. 4 step 3) and consolidation: the listed segments, a wavefront each.  Beyond MAXC candidates
// the pool is the row and the closest new edges (they arrive sorted by distance): what happens to a candidate depends on
// earlier ones only, so the result is exact if the R-th selection comes no later than the last new edge of the pool.
// lists: bit 0 / 1 = the first / second.  MAXC = 512 takes both, or the second alone, MAXC = 2,048 what it has left of the second
// (hubs: the entry point, vertices near it), and the list-based kernel the rest.  MAXC = 128 takes the first, of at most 128
// candidates, where a batch has PIVOT_MANY edges: 7 KB of LDS let 16 wavefronts into a CU for 12, below that the launch costs
// more than it gives (5 us).  100,000 points into 2 M 10.0 -> 9.8 ms; beyond, where full rows go by their memory, even.
#define PIVOT_MANY (1 << 20)
template <int S, int MAXC>
__global__ void __launch_bounds__(64, S == 1 && MAXC <= 512 ? 4 : 1) reverse_merge_u8_kernel(InsertArgs a, int lists) {
    __shared__ PivotLds<MAXC> lds;
    PivotLds<MAXC>* L = &lds;
    const int lane = lane_id(), col = lane & 31, half = lane >> 5;
    const uint32_t n1 = lists & 1 ? a.nseg[1] : 0, n = n1 + (lists & 2 ? a.nseg[2] : 0);
    const long long total = a.E ? a.E : a.B * a.R;
    for (uint32_t at = blockIdx.x; at < n; at += gridDim.x) {
        const uint64_t entry = a.lists[at < n1 ? (long long)at : total - 1 - (at - n1)];
        const uint32_t s = (uint32_t)entry;
        const uint32_t head = a.heads[s];
        if (head & 0x80000000u) continue;
        const int deg = seg_deg(entry), m = seg_new(entry);
        const long long lo = head;
        const uint32_t v = (uint32_t)(a.keys[lo] >> 32);
        uint32_t* row = a.adj + (size_t)v * a.R;
        const int mp = m < MAXC - deg ? m : MAXC - deg;
        wave_sync();  // the previous segment's reads are done
        if (deg > 0) {
            // distances of the present neighbours, then their order
            Frag<S> pv;
            pv.load(a.ds.recs + (size_t)v * a.ds.rec_stride, half, a.ds.nch);
            pv.shift();
            const int nv = frag_dot(pv, pv);
            for (int j0 = 0; j0 < deg; j0 += 32) {
                const int j = j0 + col;
                const uint32_t id = row[j < deg ? j : deg - 1];
                Frag<S> x;
                x.load(a.ds.recs + (size_t)id * a.ds.rec_stride, half, a.ds.nch);
                x.shift();
                const int d = nv + frag_dot(x, x) - 2 * frag_dot(x, pv);
                if (half == 0 && j < deg) L->raw[j] = ((uint64_t)__float_as_uint((float)(uint32_t)d) << 32) | id;
            }
            wave_sync();
            for (int j = lane; j < deg; j += 64) {
                const uint64_t k = L->raw[j];
                int place = 0;
                for (int t = 0; t < deg; t++) {
                    const uint64_t o = L->raw[t];
                    place += (o < k || (o == k && t < j)) ? 1 : 0;
                }
                L->fixed[place] = k;
                L->count[j] = 0;
            }
            wave_sync();
        }
        // both lists become one: a candidate's place is its own index and what the other list has before it
        for (int j0 = 0; j0 < mp; j0 += 64) {
            const int j = j0 + lane;
            if (j < mp) {
                const uint32_t id = a.vals[lo + j], db = (uint32_t)a.keys[lo + j];
                const uint64_t k = ((uint64_t)db << 32) | id;
                int b = 0, e = deg;
                while (b < e) {
                    const int mid = (b + e) >> 1;
                    if (L->fixed[mid] <= k) b = mid + 1;
                    else e = mid;
                }
                L->id[j + b] = id;
                L->dx[j + b] = __uint_as_float(db);
                if (b < deg) atomicAdd(&L->count[b], 1u);  // it comes before present neighbour b and later ones
            }
        }
        wave_sync();
        uint32_t before = 0;
        for (int j0 = 0; j0 < deg; j0 += 64) {
            const int j = j0 + lane;
            uint32_t c = j < deg ? L->count[j] : 0u;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl_up(c, d, 64);
                if (lane >= d) c += o;
            }
            c += before;
            before = readlane32(c, 63);
            if (j < deg) {
                const uint64_t k = L->fixed[j];
                L->id[j + c] = (uint32_t)k;
                L->dx[j + c] = __uint_as_float((uint32_t)(k >> 32));
            }
        }
        wave_sync();
        const int nsel = pivot_prune<S, MAXC>(L, a.ds.recs, (size_t)a.ds.rec_stride, a.ds.nch, deg + mp, v, a.R, a.alpha);
        wave_sync();
        if (mp < m) {
            const uint64_t tau = ((uint64_t)(uint32_t)a.keys[lo + mp - 1] << 32) | a.vals[lo + mp - 1];
            if (nsel < a.R || (((uint64_t)L->sel_dist[nsel - 1] << 32) | L->sel_id[nsel - 1]) > tau) continue;
        }
        for (int j = lane; j < a.R; j += 64) row[j] = j < nsel ? L->sel_id[j] : JX_NONE_ID;
        if (lane == 0) {
            a.clean[v] = (uint8_t)(nsel < 255 ? nsel : 255);
            const_cast<uint32_t*>(a.heads)[s] = (uint32_t)lo | 0x80000000u;
        }
    }
}

hipError_t launch_forward_prune_u8(const InsertArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)a.B), block(64);
    if (a.ds.nch <= 8) {
        if (a.L <= 128)
            hipLaunchKernelGGL((forward_prune_u8_kernel<1, 128>), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((forward_prune_u8_kernel<1, 512>), grid, block, 0, st, a);
    } else {
        if (a.L <= 128)
            hipLaunchKernelGGL((forward_prune_u8_kernel<2, 128>), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((forward_prune_u8_kernel<2, 512>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_reverse_merge_u8(const InsertArgs& a, hipStream_t st) {
    const long long most = a.E ? a.E : a.B * a.R;  // segments there can be; persistent wavefronts
    const bool many = most >= PIVOT_MANY;
    const int rest = many ? 2 : 3;
    hipError_t e = launch_reverse_class(a, many ? 128 : 512, JX_MAX_R, st);
    if (e != hipSuccess) return e;
    if (a.fresh) {
        const dim3 grid((unsigned)(most < 16384 ? most : 16384));
        if (a.ds.nch <= 8) hipLaunchKernelGGL(reverse_merge_fresh_u8_kernel<1>, grid, dim3(64), 0, st, a);
        else hipLaunchKernelGGL(reverse_merge_fresh_u8_kernel<2>, grid, dim3(64), 0, st, a);
    }
    const dim3 block(64), grid((unsigned)(most < 8192 ? most : 8192)), few((unsigned)(most < 1024 ? most : 1024));
    if (a.ds.nch <= 8) {
        if (many) hipLaunchKernelGGL((reverse_merge_u8_kernel<1, 128>), grid, block, 0, st, a, 1);
        hipLaunchKernelGGL((reverse_merge_u8_kernel<1, 512>), grid, block, 0, st, a, rest);
        if (segment_most(a) > 512) hipLaunchKernelGGL((reverse_merge_u8_kernel<1, 2048>), few, block, 0, st, a, 2);
    } else {
        if (many) hipLaunchKernelGGL((reverse_merge_u8_kernel<2, 128>), grid, block, 0, st, a, 1);
        hipLaunchKernelGGL((reverse_merge_u8_kernel<2, 512>), grid, block, 0, st, a, rest);
        if (segment_most(a) > 512) hipLaunchKernelGGL((reverse_merge_u8_kernel<2, 2048>), few, block, 0, st, a, 2);
    }
    return hipGetLastError();
}

}  // namespace jx
