// Batch insertion (Alg. 4 with the changes of Sec. 4.3 / 4.5): everything that
// follows the candidate search.
//
//   entry point   : column means (two-stage, fixed order, double) and the
//                   point nearest to the mean
//   forward prune : one wavefront per new point runs robustPrune (Alg. 3) on
//                   its final frontier, writes adjacency row, emits reverse
//                   edges (target, distance, source) to the kept neighbours only
//   sort          : stable LSD radix sort (8-bit digits) of the unified edge
//                   buffer on the 64-bit key (target << 32 | distance bits);
//                   stability leaves equal keys in emission order = ascending
//                   source id, so the order is (target, distance, source)
//   reverse merge : one wavefront per touched target: append if the row still
//                   fits, else robustPrune(row U new edges) with the existing
//                   neighbours' distances recomputed.  A row is written by
//                   exactly one wavefront: no locks (Sec. 3.3).
//
// robustPrune walks two sorted lists -- the target's existing neighbours (LDS)
// and the new candidates (global memory, already sorted) -- as one merged
// sequence.  Each time the closest live candidate p* is selected, all remaining
// live candidates p' get d(p*,p') computed (T lanes per vector, as in
// beamSearch) and are discarded when alpha * d(p*,p') <= d(p,p'), evaluated in
// float32 as one multiply and one compare.
#include "jx_distance.h"

namespace jx {

#ifndef INS_WPB
#define INS_WPB 1      // wavefronts per workgroup (they never cooperate: a slot is free as soon as its wavefront ends)
#endif
#define INS_RA JX_MAX_R

// ------------------------------------------------------------------ entry point

template <int DT>
__device__ __forceinline__ double elem_f64(const void* vecs, size_t i) {
    if (DT == JX_U8) return (double)reinterpret_cast<const uint8_t*>(vecs)[i];
    if (DT == JX_F16) return (double)(float)reinterpret_cast<const _Float16*>(vecs)[i];
    return (double)reinterpret_cast<const float*>(vecs)[i];
}

template <int DT>
__global__ void __launch_bounds__(256) col_partial_kernel(const void* vecs, long long n, int d, int nblk, double* partial) {
    const long long per = (n + nblk - 1) / nblk;
    const long long r0 = (long long)blockIdx.x * per;
    const long long r1 = r0 + per < n ? r0 + per : n;
    // a block of columns for each blockIdx.y, loads eight rows ahead of the (ordered) sum: 50,000 rows of d = 960 388 -> 29 us
    const int j = blockIdx.y * 256 + threadIdx.x;
    if (j >= d) return;
    double s = 0.0;
#pragma unroll 8
    for (long long i = r0; i < r1; i++) s += elem_f64<DT>(vecs, (size_t)i * d + j);
    partial[(size_t)blockIdx.x * d + j] = s;
}

__global__ void mean_finalize_kernel(const double* partial, int nblk, int d, long long n, float* mean) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= d) return;
    double s = 0.0;
#pragma unroll 16
    for (int b = 0; b < nblk; b++) s += partial[(size_t)b * d + j];
    mean[j] = (float)(s / (double)n);
}

template <int DT>
__global__ void __launch_bounds__(256) dist_to_mean_kernel(const void* vecs, long long n, int d, const float* mean, double* out) {
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int lane = lane_id();
    double s = 0.0;
    for (int j = lane; j < d; j += 64) {
        double v = elem_f64<DT>(vecs, (size_t)i * d + j);
        double t = v - (double)mean[j];
        s += t * t;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s += shfl_xor(s, m);
    if (lane == 0) out[i] = s;
}

// single workgroup: smallest (distance, id)
__global__ void __launch_bounds__(1024) argmin_kernel(const double* dist, long long n, uint32_t* out_id) {
    __shared__ double sd[1024];
    __shared__ long long si[1024];
    double bd = __builtin_inf();
    long long bi = 0x7FFFFFFFFFFFFFFFLL;
    for (long long i = threadIdx.x; i < n; i += 1024) {
        double v = dist[i];
        if (v < bd || (v == bd && i < bi)) {
            bd = v;
            bi = i;
        }
    }
    sd[threadIdx.x] = bd;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            double od = sd[threadIdx.x + s];
            long long oi = si[threadIdx.x + s];
            if (od < sd[threadIdx.x] || (od == sd[threadIdx.x] && oi < si[threadIdx.x])) {
                sd[threadIdx.x] = od;
                si[threadIdx.x] = oi;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *out_id = (uint32_t)si[0];
}

// ------------------------------------------------------------------ robustPrune

struct PruneLds {
    uint64_t a_key[INS_RA];   // existing neighbours sorted by (distance, id); key = distance bits << 32 | id
    uint64_t a_tmp[INS_RA];
    uint64_t cand_key[64];
    uint32_t cand_id[64];
    uint32_t cand_src[64];
    uint32_t sel_id[INS_RA];
    uint32_t sel_dist[INS_RA];
    uint8_t a_dead[INS_RA];
};

template <int KIND>
__device__ __forceinline__ float code_to_dist(uint32_t code) {
    if constexpr (KIND == K_U8)
        return (float)code;
    else
        return ordered_to_f32(code);
}

// Candidate list B in global memory: ids and non-negative float distance bits
// with element strides, plus one discard byte per element.
struct BList {
    const uint32_t* ids;
    const uint32_t* dbits;
    int id_stride, d_stride;
    int n;
    uint8_t* dead;
};

// Evaluate d(pivot, c) for the live elements of one 64-wide chunk and discard
// those with alpha * d(pivot,c) <= d(p,c).
// CACHED: the candidates' vectors sit in an LDS cache, slot i = position i of
// list A; the record "id" handed to the distance provider is then the slot.
template <int KIND, int T, int CPL, bool IS_A, bool CACHED = false>
__device__ __forceinline__ void kill_chunk(const QueryRegs<KIND, CPL, 0>& q, const DistSrc& ds, PruneLds* L, const BList& B,
                                           int c0, int n, float alpha, int g, int lig, int lane) {
    constexpr int G = 64 / T;
    constexpr int U0 = (8 / CPL) > 0 ? (8 / CPL) : 1;
    constexpr int U = U0 < (64 / G) ? U0 : (64 / G);
    const int i = c0 + lane;
    bool alive = false;
    uint32_t id = JX_NONE_ID;
    if (i < n) {
        if (IS_A) {
            alive = L->a_dead[i] == 0;
            id = CACHED ? (uint32_t)i : (uint32_t)L->a_key[i];
        } else {
            alive = B.dead[i] == 0;
            id = B.ids[(size_t)i * B.id_stride];
        }
    }
    const uint64_t am = ballot(alive);
    const int n_alive = __builtin_popcountll(am);
    if (n_alive == 0) return;
    if (alive) {
        int slot = prefix_count(am);
        L->cand_id[slot] = id;
        L->cand_src[slot] = (uint32_t)i;
    }
    wave_sync();
    for (int s0 = 0; s0 < n_alive; s0 += G * U)
        eval_batch<KIND, T, CPL, 0, U>(q, ds, s0, n_alive, L->cand_id, L->cand_key, g, lig);
    wave_sync();
    if (lane < n_alive) {
        const uint32_t src = L->cand_src[lane];
        const float d1 = code_to_dist<KIND>(key_dist(L->cand_key[lane]));
        float d2;
        if (IS_A)
            d2 = __uint_as_float((uint32_t)(L->a_key[src] >> 32));
        else
            d2 = __uint_as_float(B.dbits[(size_t)src * B.d_stride]);
        if (__fmul_rn(alpha, d1) <= d2) {
            if (IS_A)
                L->a_dead[src] = 1;
            else
                B.dead[src] = 1;
        }
    }
    __threadfence_block();
    wave_sync();
}

// Alg. 3 over the merged sequence of A (LDS, nA entries) and B.  Returns the
// number of selected ids (L->sel_id / L->sel_dist, selection order).
template <int KIND, int T, int CPL, bool CACHED = false>
__device__ __forceinline__ int robust_prune_wave(const DistSrc& ds, PruneLds* L, int nA, const BList& B, int R, float alpha) {
    const int lane = lane_id();
    const int g = lane / T, lig = lane % T;
    int iA = 0, iB = 0, nsel = 0;
    QueryRegs<KIND, CPL, 0> q;
    while (nsel < R) {
        while (iA < nA && L->a_dead[iA]) iA++;
        while (iB < B.n) {
            const int i = iB + lane;
            const bool alive = i < B.n && B.dead[i] == 0;
            const uint64_t m = ballot(alive);
            if (m) {
                iB += __builtin_ctzll(m);
                break;
            }
            iB += 64;
        }
        const bool hasA = iA < nA, hasB = iB < B.n;
        if (!hasA && !hasB) break;
        uint64_t kA = JX_EMPTY_KEY, kB = JX_EMPTY_KEY;
        if (hasA) kA = L->a_key[iA];
        if (hasB) kB = ((uint64_t)B.dbits[(size_t)iB * B.d_stride] << 32) | B.ids[(size_t)iB * B.id_stride];
        const bool takeA = kA < kB;
        const uint64_t kp = takeA ? kA : kB;
        const uint32_t pid = (CACHED && takeA) ? (uint32_t)iA : (uint32_t)kp;  // record to load as the pivot
        if (takeA) iA++; else iB++;
        if (lane == 0) {
            L->sel_id[nsel] = (uint32_t)kp;
            L->sel_dist[nsel] = (uint32_t)(kp >> 32);
        }
        nsel++;
        if (nsel >= R) break;
        load_query<KIND, T, CPL, 0>(q, ds, (int64_t)pid, lig);
        for (int c0 = iA; c0 < nA; c0 += 64) kill_chunk<KIND, T, CPL, true, CACHED>(q, ds, L, B, c0, nA, alpha, g, lig, lane);
        for (int c0 = iB; c0 < B.n; c0 += 64) kill_chunk<KIND, T, CPL, false, false>(q, ds, L, B, c0, B.n, alpha, g, lig, lane);
    }
    wave_sync();
    return nsel;
}

template <int KIND, int T, int CPL>
__global__ void __launch_bounds__(INS_WPB * 64) forward_prune_kernel(InsertArgs a) {
    __shared__ PruneLds lds[INS_WPB];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const long long i = (long long)blockIdx.x * INS_WPB + wave;
    if (i >= a.B) return;
    PruneLds* L = &lds[wave];
    long long xid = a.id_base + i;
    if (xid >= a.id_skip) xid++;
    BList B;
    B.ids = a.cand_ids + (size_t)i * a.L;
    B.dbits = a.cand_dist + (size_t)i * a.L;
    B.id_stride = 1;
    B.d_stride = 1;
    B.dead = a.dead + (size_t)i * a.L;
    // lists longer than 128: the block-row Gram-matrix kernel has run first and marks what it has done
    if (a.gram && a.L > 128 && B.dead[0] == 0xFF) return;
    // the frontier is filled from the left: count its valid entries
    int nB = 0;
    for (int c0 = 0; c0 < a.L; c0 += 64) {
        const int j = c0 + lane;
        const bool valid = j < a.L && B.ids[j] != JX_NONE_ID;
        if (j < a.L) B.dead[j] = 0;
        nB += __builtin_popcountll(ballot(valid));
    }
    B.n = nB;
    if (a.gram && nB <= 128) return;  // served by the Gram-matrix kernel
    __threadfence_block();
    wave_sync();
    const int nsel = robust_prune_wave<KIND, T, CPL>(a.ds, L, 0, B, a.R, a.alpha);
    if (KIND == K_U8 && lane == 0) a.clean[xid] = (uint8_t)(nsel < 255 ? nsel : 255);
    uint32_t* row = a.adj + (size_t)xid * a.R;
    for (int j = lane; j < a.R; j += 64) {
        const bool on = j < nsel;
        const uint32_t v = on ? L->sel_id[j] : JX_NONE_ID;
        row[j] = v;
        a.keys[(size_t)i * a.R + j] = on ? (((uint64_t)v << 32) | L->sel_dist[j]) : JX_EMPTY_KEY;
        a.vals[(size_t)i * a.R + j] = on ? (uint32_t)xid : JX_NONE_ID;
    }
}

template <int KIND, int T, int CPL>
__global__ void __launch_bounds__(INS_WPB * 64) reverse_merge_kernel(InsertArgs a) {
    __shared__ PruneLds lds[INS_WPB];
    constexpr int G = 64 / T;
    constexpr int U0 = (8 / CPL) > 0 ? (8 / CPL) : 1;
    constexpr int U = U0 < (64 / G) ? U0 : (64 / G);
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int g = lane / T, lig = lane % T;
    PruneLds* L = &lds[wave];
    extern __shared__ __align__(16) unsigned char vcache[];  // INS_WPB x vec_cache_bytes
    const long long nseg = *a.nseg;
    const long long total = a.E ? a.E : a.B * a.R;
    for (long long s = (long long)blockIdx.x * INS_WPB + wave; s < nseg; s += (long long)gridDim.x * INS_WPB) {
        const uint32_t head = a.heads[s];
        if (head & 0x80000000u) continue;  // merged by the Gram-matrix kernel, which marks what it has done
        const long long lo = head;
        const uint32_t v = (uint32_t)(a.keys[lo] >> 32);
        if (v == JX_NONE_ID) continue;  // tail of empty keys
        // segment length
        int m = 0;
        for (long long c0 = lo; c0 < total; c0 += 64) {
            const long long j = c0 + lane;
            const bool same = j < total && (uint32_t)(a.keys[j] >> 32) == v;
            const uint64_t sm = ballot(same);
            m += __builtin_popcountll(sm);
            if (sm != ~0ull) break;
        }
        uint32_t* row = a.adj + (size_t)v * a.R;
        int deg = 0;
        for (int rb = 0; rb < a.R; rb += 64) {
            const bool on = rb + lane < a.R && row[rb + lane] != JX_NONE_ID;
            deg += __builtin_popcountll(ballot(on));
        }
        if (a.force_prune) deg = 0;  // consolidation: the segment holds the whole candidate set
        if (!a.force_prune && deg + m <= a.R) {
            for (int j = lane; j < m; j += 64) row[deg + j] = a.vals[lo + j];
            continue;
        }
        // distances from v to its existing neighbours, then sort them
        QueryRegs<KIND, CPL, 0> q;
        load_query<KIND, T, CPL, 0>(q, a.ds, (int64_t)v, lig);
        for (int c0 = 0; c0 < deg; c0 += 64) {
            const int nn = deg - c0 < 64 ? deg - c0 : 64;
            if (lane < nn) L->cand_id[lane] = row[c0 + lane];
            wave_sync();
            for (int s0 = 0; s0 < nn; s0 += G * U)
                eval_batch<KIND, T, CPL, 0, U>(q, a.ds, s0, nn, L->cand_id, L->cand_key, g, lig);
            wave_sync();
            if (lane < nn) {
                const uint64_t k = L->cand_key[lane];
                const float dd = code_to_dist<KIND>(key_dist(k));
                L->a_tmp[c0 + lane] = ((uint64_t)__float_as_uint(dd) << 32) | (uint64_t)key_id(k);
            }
            wave_sync();
        }
        // Small case (the usual one: a full row plus a few new edges): merge both
        // lists into one, pull all candidate vectors into LDS once, and run the
        // selection loop on the cache -- no global load on its critical path.
        const int M = deg + m;
        const bool cached = M <= INS_RA && (long long)M * a.ds.rec_stride <= a.vec_cache_bytes;
        if (cached) {
            for (int j = lane; j < m; j += 64)
                L->a_tmp[deg + j] = ((uint64_t)reinterpret_cast<const uint32_t*>(a.keys + lo + j)[0] << 32) | a.vals[lo + j];
            wave_sync();
        }
        const int nsort = cached ? M : deg;
        for (int j = lane; j < nsort; j += 64) {
            const uint64_t k = L->a_tmp[j];
            int rank = 0;
            for (int t = 0; t < nsort; t++) rank += (L->a_tmp[t] < k) ? 1 : 0;
            L->a_key[rank] = k;
            L->a_dead[j] = 0;
        }
        int nsel;
        if (cached) {
            wave_sync();
            unsigned char* vc = vcache + (size_t)wave * a.vec_cache_bytes;
            const int nch = a.ds.nch;
            for (int c = lane; c < M * nch; c += 64) {
                const int sl = c / nch, ch = c - sl * nch;
                const uint32_t id = (uint32_t)L->a_key[sl];
                *reinterpret_cast<uint4*>(vc + (size_t)sl * a.ds.rec_stride + ch * 16) =
                    load16(a.ds.recs + (size_t)id * (size_t)a.ds.rec_stride + (size_t)ch * 16);
            }
            DistSrc cds = a.ds;
            cds.recs = vc;
            cds.qrecs = vc;
            BList none;
            none.ids = nullptr;
            none.dbits = nullptr;
            none.id_stride = none.d_stride = 1;
            none.n = 0;
            none.dead = nullptr;
            __threadfence_block();
            wave_sync();
            nsel = robust_prune_wave<KIND, T, CPL, true>(cds, L, M, none, a.R, a.alpha);
        } else {
            BList B;
            B.ids = a.vals + lo;
            B.dbits = reinterpret_cast<const uint32_t*>(a.keys + lo);
            B.id_stride = 1;
            B.d_stride = 2;
            B.dead = a.dead + lo;
            // A hub (the entry point, vertices near it) can receive thousands of reverse edges in one batch, and every
            // selection of the loop below passes over all live candidates.  Alg. 3 visits candidates in (distance, id)
            // order, stops at R selections, and what happens to a candidate depends on earlier ones only: prune a
            // prefix of the sorted new edges first; if the R-th selection comes no later than the last included new
            // edge, the excluded ones could not have mattered and the result is exact.  Otherwise take four times as many.
            int mp = m < 512 ? m : 512;
            for (;;) {
                B.n = mp;
                for (int j = lane; j < mp; j += 64) B.dead[j] = 0;
                for (int j = lane; j < deg; j += 64) L->a_dead[j] = 0;
                __threadfence_block();
                wave_sync();
                nsel = robust_prune_wave<KIND, T, CPL, false>(a.ds, L, deg, B, a.R, a.alpha);
                if (mp == m) break;
                const uint64_t tau = ((uint64_t)B.dbits[(size_t)(mp - 1) * 2] << 32) | B.ids[mp - 1];
                if (nsel >= a.R && (((uint64_t)L->sel_dist[nsel - 1] << 32) | L->sel_id[nsel - 1]) <= tau) break;
                mp = (long long)mp * 4 < m ? mp * 4 : m;
            }
        }
        for (int j = lane; j < a.R; j += 64) row[j] = j < nsel ? L->sel_id[j] : JX_NONE_ID;
        if (KIND == K_U8 && lane == 0) a.clean[v] = (uint8_t)(nsel < 255 ? nsel : 255);
        wave_sync();
    }
}

// ------------------------------------------------------------------ radix sort

#define RS_ITEMS 16
#define RS_TILE (256 * RS_ITEMS)

// exclusive prefix sum of `total` counters, single workgroup: 1,024 consecutive ones per wavefront and round (one per thread
// took a microsecond for every 1,024: 200,000 flags of a compaction 209 -> 75 us)
__global__ void __launch_bounds__(1024) radix_scan_kernel(uint32_t* table, long long total) {
    __shared__ uint32_t ws[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (long long c0 = 0; c0 < total; c0 += 16384) {
        const long long i0 = c0 + (long long)wave * 1024 + lane;
        uint32_t v[16], x[16], sum = 0;
#pragma unroll
        for (int e = 0; e < 16; e++) v[e] = i0 + 64 * e < total ? table[i0 + 64 * e] : 0u;
#pragma unroll
        for (int e = 0; e < 16; e++) {
            x[e] = v[e];
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const uint32_t o = __shfl_up(x[e], s, 64);
                if (lane >= s) x[e] += o;
            }
        }
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const uint32_t row = readlane32(x[e], 63);
            x[e] += sum - v[e];
            sum += row;
        }
        if (lane == 0) ws[wave] = sum;
        __syncthreads();
        uint32_t at = carry, all = 0;
#pragma unroll
        for (int w = 0; w < 16; w++) {
            const uint32_t t = ws[w];
            at += w < wave ? t : 0u;
            all += t;
        }
        carry += all;
#pragma unroll
        for (int e = 0; e < 16; e++)
            if (i0 + 64 * e < total) table[i0 + 64 * e] = at + x[e];
        __syncthreads();
    }
}

// 8-bit digits.  A tile of 4,096 keys is sorted on the digit inside LDS by two stable 4-bit passes (every thread
// counts the 16 keys it holds per nibble value; an exclusive scan over the counters in nibble-major, thread-minor
// order gives each key its rank), then written out run by run.
__global__ void __launch_bounds__(256) radix_hist8_kernel(const uint64_t* keys, long long n, int shift, uint32_t* table, int ntiles) {
    __shared__ uint32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const long long base = (long long)blockIdx.x * RS_TILE;
#pragma unroll
    for (int e = 0; e < RS_ITEMS; e++) {
        const long long i = base + e * 256 + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 255], 1u);
    }
    __syncthreads();
    table[(size_t)threadIdx.x * ntiles + blockIdx.x] = cnt[threadIdx.x];
}

// one workgroup per digit: exclusive prefix sum over the tiles of its row, row total to table[256 * ntiles + digit]
__global__ void __launch_bounds__(1024) radix_rowscan8_kernel(uint32_t* table, int ntiles) {
    __shared__ uint32_t ws[16];
    __shared__ uint32_t carry_s;
    uint32_t* row = table + (size_t)blockIdx.x * ntiles;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c0 = 0; c0 < ntiles; c0 += 1024) {
        const int i = c0 + threadIdx.x;
        const uint32_t v = i < ntiles ? row[i] : 0u;
        uint32_t x = v;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            uint32_t o = __shfl_up(x, s, 64);
            if (lane >= s) x += o;
        }
        if (lane == 63) ws[wave] = x;
        __syncthreads();
        uint32_t woff = 0;
        for (int w = 0; w < wave; w++) woff += ws[w];
        const uint32_t carry = carry_s;
        if (i < ntiles) row[i] = carry + woff + x - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry_s = carry + woff + x;
        __syncthreads();
    }
    if (threadIdx.x == 0) table[(size_t)256 * ntiles + blockIdx.x] = carry_s;
}

// exclusive scan of psum[256] in place by the first wavefront (4 entries per lane); callers synchronise around it
__device__ __forceinline__ void scan256_wave0(uint32_t* psum, int t) {
    if (t < 64) {
        uint32_t a0 = psum[4 * t], a1 = psum[4 * t + 1], a2 = psum[4 * t + 2], a3 = psum[4 * t + 3];
        uint32_t tot = a0 + a1 + a2 + a3, x = tot;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            uint32_t o = __shfl_up(x, s, 64);
            if (t >= s) x += o;
        }
        uint32_t ex = x - tot;
        psum[4 * t] = ex;
        psum[4 * t + 1] = ex + a0;
        psum[4 * t + 2] = ex + a0 + a1;
        psum[4 * t + 3] = ex + a0 + a1 + a2;
    }
}

__global__ void __launch_bounds__(256) radix_scatter8_kernel(const uint64_t* keys, const uint32_t* vals, uint64_t* keys_out,
                                                            uint32_t* vals_out, long long n, int shift,
                                                            const uint32_t* table, int ntiles) {
    __shared__ uint64_t sk[RS_TILE];
    __shared__ uint32_t sv[RS_TILE];
    __shared__ uint16_t hist[16 * 256];  // [digit][thread]
    __shared__ uint32_t psum[256];
    __shared__ uint32_t gbase[256];
    __shared__ uint16_t dstart[256];
    const int t = threadIdx.x;
    const long long tile0 = (long long)blockIdx.x * RS_TILE;
    const int cnt = (int)(n - tile0 < (long long)RS_TILE ? n - tile0 : (long long)RS_TILE);
    // where each digit's run of this tile starts in the output: digits below it, then the tiles before this one
    psum[t] = table[(size_t)256 * ntiles + t];
    __syncthreads();
    scan256_wave0(psum, t);
    __syncthreads();
    gbase[t] = psum[t] + table[(size_t)t * ntiles + blockIdx.x];
    uint64_t k[RS_ITEMS];
    uint32_t v[RS_ITEMS];
#pragma unroll
    for (int e = 0; e < RS_ITEMS; e++) {
        const long long i = tile0 + (long long)t * RS_ITEMS + e;
        k[e] = i < n ? keys[i] : JX_EMPTY_KEY;  // padding carries the largest digit and comes last in the tile: it stays last
        v[e] = i < n ? vals[i] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; half++) {
        const int sh = shift + 4 * half;
#pragma unroll
        for (int d = 0; d < 16; d++) hist[d * 256 + t] = 0;
#pragma unroll
        for (int e = 0; e < RS_ITEMS; e++) hist[((k[e] >> sh) & 15) * 256 + t]++;
        __syncthreads();
        uint32_t loc[16];
        uint32_t sum = 0;
#pragma unroll
        for (int e = 0; e < 16; e++) {
            loc[e] = sum;
            sum += hist[t * 16 + e];
        }
        psum[t] = sum;
        __syncthreads();
        scan256_wave0(psum, t);
        __syncthreads();
        const uint32_t off = psum[t];
#pragma unroll
        for (int e = 0; e < 16; e++) hist[t * 16 + e] = (uint16_t)(off + loc[e]);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < RS_ITEMS; e++) {
            const int d = (int)((k[e] >> sh) & 15);
            const uint32_t r = hist[d * 256 + t];
            hist[d * 256 + t] = (uint16_t)(r + 1);
            sk[r] = k[e];
            sv[r] = v[e];
        }
        __syncthreads();
        if (half == 0) {
#pragma unroll
            for (int e = 0; e < RS_ITEMS; e++) {
                k[e] = sk[t * RS_ITEMS + e];
                v[e] = sv[t * RS_ITEMS + e];
            }
            __syncthreads();
        }
    }
    for (int i = t; i < cnt; i += 256) {
        const int d = (int)((sk[i] >> shift) & 255);
        if (i == 0 || (int)((sk[i - 1] >> shift) & 255) != d) dstart[d] = (uint16_t)i;
    }
    __syncthreads();
    for (int i = t; i < cnt; i += 256) {
        const uint64_t key = sk[i];
        const int d = (int)((key >> shift) & 255);
        const size_t pos = (size_t)gbase[d] + (size_t)(i - dstart[d]);
        keys_out[pos] = key;
        vals_out[pos] = sv[i];
    }
}

// ---- small edge buffers: chunks sorted by a workgroup each, then merge passes
//
// A pass of the radix sort is three launches of 4 to 14 us however few the keys are, and a sort is six or eight passes:
// most of an insertion of a few points.  Up to SORT_ONE pairs are sorted by one workgroup, which lists the segments as well;
// up to SORT_MERGE pairs by a workgroup per SORT_CHUNK pairs and a launch per eightfold of the runs, every pair
// finding its place by binary searches in up to seven neighbouring runs.  The order is (key, value): what the stable radix sort
// gives, because equal keys are emitted in ascending order of their values.
// A chunk is a bitonic network over V pairs per thread in registers: strides below V are moves inside a thread, those below
// 64 V go from lane to lane, and only the few that are wider through LDS with a barrier.  With every stride through LDS
// 4,096 pairs took 53 us, now 28; 2,048 27.8 and 17, 20,000 80 and 43, 600,000 188 and 163.  Chunks of 2,048: two of them and a
// merge are done before one workgroup has sorted 8,192 (55 us).  Beyond 2^20 the radix sort takes over: 2.4 M pairs 478 us,
// 626 by merges.
#define SORT_ONE 4096
#define SORT_CHUNK 2048  // 4,096 beyond 2^18 pairs, where the last pass merges four runs instead of eight: 2^20 pairs 252 us -> 220
#define SORT_MERGE (1 << 20)

__device__ __forceinline__ bool pair_after(uint64_t a, uint32_t x, uint64_t b, uint32_t y) { return a > b || (a == b && x > y); }

// one stage of the network: pair i = tid V + r against pair i ^ J, ascending where i & K is 0, and the stages that follow
template <int T, int V, int K, int J>
__device__ __forceinline__ void sort_pairs(uint64_t (&k)[V], uint32_t (&v)[V], uint64_t* sk, uint32_t* sv, const int tid) {
    if constexpr (J < V) {
#pragma unroll
        for (int r = 0; r < V; r++)
            if ((r & J) == 0) {
                const bool up = K < V ? (r & K) == 0 : (tid & (K / V)) == 0;
                const uint64_t a = k[r], b = k[r | J];
                const uint32_t x = v[r], y = v[r | J];
                const bool swap = pair_after(a, x, b, y) == up;
                k[r] = swap ? b : a;
                k[r | J] = swap ? a : b;
                v[r] = swap ? y : x;
                v[r | J] = swap ? x : y;
            }
    } else {
        const bool low = ((tid & (J / V)) == 0) == ((tid & (K / V)) == 0);  // keeps the smaller one
        if constexpr (J / V >= 64) {  // another wavefront's
            __syncthreads();  // what was read last is no longer needed
#pragma unroll
            for (int r = 0; r < V; r++) {
                sk[r * T + tid] = k[r];
                sv[r * T + tid] = v[r];
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < V; r++) {
            uint64_t b;
            uint32_t y;
            if constexpr (J / V < 64) {
                b = (uint64_t)lane_xor_u32<J / V>((uint32_t)(k[r] >> 32)) << 32 | lane_xor_u32<J / V>((uint32_t)k[r]);
                y = lane_xor_u32<J / V>(v[r]);
            } else {
                b = sk[r * T + (tid ^ (J / V))];
                y = sv[r * T + (tid ^ (J / V))];
            }
            const bool take = pair_after(k[r], v[r], b, y) == low;
            k[r] = take ? b : k[r];
            v[r] = take ? y : v[r];
        }
    }
    if constexpr (J > 1)
        sort_pairs<T, V, K, J / 2>(k, v, sk, sv, tid);
    else if constexpr (K < T * V)
        sort_pairs<T, V, K * 2, K>(k, v, sk, sv, tid);
}

// one workgroup per T V pairs; heads / counters: NULL, or the segment list of a single chunk
template <int T, int V>
__global__ void __launch_bounds__(T) sort_chunk_kernel(const uint64_t* keys, const uint32_t* vals, uint64_t* keys_out, uint32_t* vals_out,
                                                      long long n, uint32_t* heads, uint32_t* counters) {
    extern __shared__ __align__(16) unsigned char dyn[];
    uint64_t* sk = reinterpret_cast<uint64_t*>(dyn);          // [T V]
    uint32_t* sv = reinterpret_cast<uint32_t*>(sk + T * V);   // [T V]
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long base = (long long)blockIdx.x * (T * V);
    const int m = (int)(n - base < T * V ? n - base : T * V);
    {
        uint64_t k[V];
        uint32_t v[V];
#pragma unroll
        for (int r = 0; r < V; r++) {
            const int i = r * T + tid;
            k[r] = i < m ? keys[base + i] : JX_EMPTY_KEY;
            v[r] = i < m ? vals[base + i] : JX_NONE_ID;
        }
        sort_pairs<T, V, 2, 1>(k, v, sk, sv, tid);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < V; r++) {
            sk[tid * V + r] = k[r];
            sv[tid * V + r] = v[r];
        }
    }
    __syncthreads();
    for (int i = tid; i < m; i += T) {
        keys_out[base + i] = sk[i];
        vals_out[base + i] = sv[i];
    }
    if (!heads) return;
    uint32_t done = 0;  // heads of the pairs before this round's
    for (int i0 = 0; i0 < m; i0 += T) {
        const int i = i0 + tid;
        const uint32_t t = i < m ? (uint32_t)(sk[i] >> 32) : JX_NONE_ID;
        const bool head = t != JX_NONE_ID && (i == 0 || (uint32_t)(sk[i - 1] >> 32) != t);
        const uint64_t hm = ballot(head);
        if (lane == 0) wsum[wave] = (uint32_t)__builtin_popcountll(hm);
        __syncthreads();
        uint32_t before = done, all = 0;
        for (int w = 0; w < T / 64; w++) {
            before += w < wave ? wsum[w] : 0u;
            all += wsum[w];
        }
        if (head) heads[before + (uint32_t)prefix_count(hm)] = (uint32_t)i;
        done += all;
        __syncthreads();
    }
    if (tid < 16) counters[tid] = tid == 0 ? done : 0u;
}

template <int T, int V>
static hipError_t launch_sort_chunk(const uint64_t* keys, const uint32_t* vals, uint64_t* keys_out, uint32_t* vals_out, long long n,
                                    uint32_t* heads, uint32_t* counters, hipStream_t st) {
    const size_t sh = (size_t)T * V * 12;  // at most 48 KB
    hipLaunchKernelGGL((sort_chunk_kernel<T, V>), dim3((unsigned)((n + T * V - 1) / (T * V))), dim3(T), sh, st, keys, vals, keys_out, vals_out, n,
                       heads, counters);
    return hipGetLastError();
}

// sorted runs of `run` pairs (a power of two, at least 256) -> runs of WAYS times as many
template <int WAYS>
__global__ void __launch_bounds__(256) merge_runs_kernel(const uint64_t* keys, const uint32_t* vals, uint64_t* keys_out, uint32_t* vals_out,
                                                        int n, int run) {
    const int b0 = (int)blockIdx.x * 256, i = b0 + (int)threadIdx.x;
    if (i >= n) return;
    const int group = b0 / (run * WAYS) * (run * WAYS), own = (b0 - group) / run;  // the same for the whole workgroup
    const uint64_t k = keys[i];
    const uint32_t v = vals[i];
    const bool padding = k == JX_EMPTY_KEY;  // all alike: those of earlier runs come first
    int cnt[WAYS], len[WAYS];
#pragma unroll
    for (int o = 0; o < WAYS; o++) {
        const long long left = (long long)n - group - (long long)o * run;
        len[o] = o == own || left <= 0 ? 0 : left < run ? (int)left : run;
        cnt[o] = 0;
    }
    // in each run the pairs that come before this one; the loads of a step are under way together
    for (int step = run; step >= 1; step >>= 1) {
        int at[WAYS];
        uint64_t ko[WAYS];
#pragma unroll
        for (int o = 0; o < WAYS; o++) {
            at[o] = cnt[o] + step <= len[o] ? group + o * run + cnt[o] + step - 1 : 0;
            ko[o] = keys[at[o]];
        }
#pragma unroll
        for (int o = 0; o < WAYS; o++) {
            uint32_t vo = v;
            if (ko[o] == k && !padding) vo = vals[at[o]];
            const bool before = ko[o] < k || (ko[o] == k && (vo < v || (vo == v && o < own)));
            cnt[o] += (before && cnt[o] + step <= len[o]) ? step : 0;
        }
    }
    int at = i - own * run;
#pragma unroll
    for (int o = 0; o < WAYS; o++) at += cnt[o];
    keys_out[at] = k;
    vals_out[at] = v;
}

__global__ void __launch_bounds__(1024) segment_heads_kernel(const uint64_t* keys, long long n, uint32_t* heads, uint32_t* nseg) {
    __shared__ uint32_t woff[17];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    // 4 consecutive keys per thread
    const long long i0 = ((long long)blockIdx.x * 1024 + threadIdx.x) * 4;
    bool is_head[4];
    int mine = 0;
    uint32_t prev = JX_NONE_ID;
    if (i0 > 0 && i0 < n) prev = (uint32_t)(keys[i0 - 1] >> 32);
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const long long i = i0 + e;
        uint32_t t = JX_NONE_ID;
        if (i < n) t = (uint32_t)(keys[i] >> 32);
        is_head[e] = t != JX_NONE_ID && (i == 0 || t != prev);
        mine += is_head[e] ? 1 : 0;
        prev = t;
    }
    // one atomic per workgroup (same-address atomics serialise; the order of the list does not matter)
    uint32_t x = (uint32_t)mine;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        uint32_t o = __shfl_up(x, s, 64);
        if (lane >= s) x += o;
    }
    if (lane == 63) woff[wave] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0;
        for (int w = 0; w < 16; w++) {
            const uint32_t c = woff[w];
            woff[w] = tot;
            tot += c;
        }
        woff[16] = tot ? atomicAdd(nseg, tot) : 0u;
    }
    __syncthreads();
    uint32_t pos = woff[16] + woff[wave] + x - (uint32_t)mine;
#pragma unroll
    for (int e = 0; e < 4; e++)
        if (is_head[e]) heads[pos++] = (uint32_t)(i0 + e);
}

// ------------------------------------------------------------------ launchers

hipError_t launch_entry_point(const void* vecs, int dtype, long long n, int d, double* partial, float* mean, double* dist,
                              uint32_t* out_id, hipStream_t st) {
    int nblk = (int)((n + 255) / 256);
    if (nblk > 512) nblk = 512;
    if (nblk < 1) nblk = 1;
    if (dtype == JX_U8)
        hipLaunchKernelGGL(col_partial_kernel<JX_U8>, dim3(nblk, (d + 255) / 256), dim3(256), 0, st, vecs, n, d, nblk, partial);
    else if (dtype == JX_F16)
        hipLaunchKernelGGL(col_partial_kernel<JX_F16>, dim3(nblk, (d + 255) / 256), dim3(256), 0, st, vecs, n, d, nblk, partial);
    else
        hipLaunchKernelGGL(col_partial_kernel<JX_F32>, dim3(nblk, (d + 255) / 256), dim3(256), 0, st, vecs, n, d, nblk, partial);
    hipLaunchKernelGGL(mean_finalize_kernel, dim3((d + 63) / 64), dim3(64), 0, st, partial, nblk, d, n, mean);
    if (dtype == JX_U8)
        hipLaunchKernelGGL(dist_to_mean_kernel<JX_U8>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, vecs, n, d, mean, dist);
    else if (dtype == JX_F16)
        hipLaunchKernelGGL(dist_to_mean_kernel<JX_F16>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, vecs, n, d, mean, dist);
    else
        hipLaunchKernelGGL(dist_to_mean_kernel<JX_F32>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, vecs, n, d, mean, dist);
    hipLaunchKernelGGL(argmin_kernel, dim3(1), dim3(1024), 0, st, dist, n, out_id);
    return hipGetLastError();
}

// column means only (two-stage, fixed order): the RaBitQ centroid
hipError_t launch_column_mean(const void* vecs, int dtype, long long n, int d, double* partial, float* mean, hipStream_t st) {
    int nblk = (int)((n + 255) / 256);
    if (nblk > 512) nblk = 512;
    if (nblk < 1) nblk = 1;
    if (dtype == JX_U8)
        hipLaunchKernelGGL(col_partial_kernel<JX_U8>, dim3(nblk, (d + 255) / 256), dim3(256), 0, st, vecs, n, d, nblk, partial);
    else if (dtype == JX_F16)
        hipLaunchKernelGGL(col_partial_kernel<JX_F16>, dim3(nblk, (d + 255) / 256), dim3(256), 0, st, vecs, n, d, nblk, partial);
    else
        hipLaunchKernelGGL(col_partial_kernel<JX_F32>, dim3(nblk, (d + 255) / 256), dim3(256), 0, st, vecs, n, d, nblk, partial);
    hipLaunchKernelGGL(mean_finalize_kernel, dim3((d + 63) / 64), dim3(64), 0, st, partial, nblk, d, n, mean);
    return hipGetLastError();
}

int entry_point_partial_blocks(long long n) {
    long long nblk = (n + 255) / 256;
    return (int)(nblk > 512 ? 512 : (nblk < 1 ? 1 : nblk));
}

template <int KIND, int T, int CPL>
static hipError_t launch_prune_pair(bool forward, const InsertArgs& a, hipStream_t st) {
    if (forward) {
        dim3 grid((unsigned)((a.B + INS_WPB - 1) / INS_WPB));
        const size_t sh = (size_t)INS_WPB * a.vec_cache_bytes;
        if (sh > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute((const void*)forward_prune_kernel<KIND, T, CPL>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL((forward_prune_kernel<KIND, T, CPL>), grid, dim3(INS_WPB * 64), sh, st, a);
    } else {
        long long want = ((a.E ? a.E : a.B * a.R) + INS_WPB - 1) / INS_WPB;
        const long long cap = 16384 / INS_WPB;  // persistent wavefronts, segments dealt round-robin
        unsigned grid = (unsigned)(want < cap ? (want < 1 ? 1 : want) : cap);
        hipLaunchKernelGGL((reverse_merge_kernel<KIND, T, CPL>), dim3(grid), dim3(INS_WPB * 64),
                           (size_t)INS_WPB * a.vec_cache_bytes, st, a);
    }
    return hipGetLastError();
}

template <int KIND>
static hipError_t launch_prune_shape(bool forward, const InsertArgs& a, hipStream_t st) {
    // same record-to-lane mapping as beamSearch: 2 chunks per lane up to 64 chunks
    const int nch = a.ds.nch;
    if (nch <= 8) return launch_prune_pair<KIND, 4, 2>(forward, a, st);
    if (nch <= 16) return launch_prune_pair<KIND, 8, 2>(forward, a, st);
    if (nch <= 32) return launch_prune_pair<KIND, 16, 2>(forward, a, st);
    if (nch <= 64) return launch_prune_pair<KIND, 32, 2>(forward, a, st);
    if (nch <= 128) return launch_prune_pair<KIND, 64, 2>(forward, a, st);
    if (nch <= 256) return launch_prune_pair<KIND, 64, 4>(forward, a, st);
    if (nch <= 384) return launch_prune_pair<KIND, 64, 6>(forward, a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_forward_prune(int dtype, const InsertArgs& a, hipStream_t st) {
    if (a.gram == 4) return launch_forward_prune_u8(a, st);
    if (a.gram) {
        hipError_t e = launch_forward_prune_gram(dtype, a, st);
        if (e != hipSuccess || a.L <= 256) return e;  // longer lists: the list-based kernel takes the rest
    }
    if (dtype == JX_U8) return launch_prune_shape<K_U8>(true, a, st);
    if (dtype == JX_F16) return launch_prune_shape<K_F16>(true, a, st);
    return launch_prune_shape<K_F32>(true, a, st);
}

hipError_t launch_reverse_merge(int dtype, const InsertArgs& a, hipStream_t st) {
    if (a.gram) {  // then the list-based kernel: what these leave
        hipError_t e = a.gram == 4 ? launch_reverse_merge_u8(a, st) : launch_reverse_merge_gram(dtype, a, st);
        if (e != hipSuccess) return e;
        // pools of 512 (uint8) and of 256 (beside rows of at most 192) have merged every smaller segment
        if (segment_most(a) <= (a.gram == 4 ? 512 : (a.R <= 192 ? 256 : 128))) return hipSuccess;
    }
    if (dtype == JX_U8) return launch_prune_shape<K_U8>(false, a, st);
    if (dtype == JX_F16) return launch_prune_shape<K_F16>(false, a, st);
    return launch_prune_shape<K_F32>(false, a, st);
}

// Sorts n (key, value) pairs on key bits [0, nbits), stable.  The result is in keys_a / vals_a again, or where in_b is
// given, after an odd number of passes, in keys_b / vals_b (insertions into 2^16 to 2^24 points have seven: an eighth that
// moved nothing cost a build of 200,000 points 0.2 of 22.4 ms).
static hipError_t launch_radix_sort(uint64_t* keys_a, uint32_t* vals_a, uint64_t* keys_b, uint32_t* vals_b, long long n, int nbits,
                                    int low_bits, uint32_t* table, bool* in_b, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int ntiles = (int)((n + RS_TILE - 1) / RS_TILE);
    // 8-bit passes.  With 4-bit digits the same sort took 14
    // passes of 162 us at 6.4M keys; these take 80 us each: the tile leaves LDS sorted, so the global writes are runs.
    // Bits low_bits..31 are zero: no pass over them (the (vertex, candidate) pairs of a consolidation: six passes for eight)
    int shifts[9], passes = 0;
    for (int b = 0; b < (low_bits < 32 ? low_bits : 32) && b < nbits; b += 8) shifts[passes++] = b;
    for (int b = 32; b < nbits; b += 8) shifts[passes++] = b;
    if (in_b) {
        *in_b = passes & 1;
    } else if (passes & 1) {
        shifts[passes] = shifts[passes - 1];  // the same digit again moves nothing
        passes++;
    }
    uint64_t *ki = keys_a, *ko = keys_b;
    uint32_t *vi = vals_a, *vo = vals_b;
    for (int p = 0; p < passes; p++) {
        const int shift = shifts[p];
        hipLaunchKernelGGL(radix_hist8_kernel, dim3(ntiles), dim3(256), 0, st, ki, n, shift, table, ntiles);
        hipLaunchKernelGGL(radix_rowscan8_kernel, dim3(256), dim3(1024), 0, st, table, ntiles);
        hipLaunchKernelGGL(radix_scatter8_kernel, dim3(ntiles), dim3(256), 0, st, ki, vi, ko, vo, n, shift, table, ntiles);
        uint64_t* tk = ki; ki = ko; ko = tk;
        uint32_t* tv = vi; vi = vo; vo = tv;
    }
    return hipGetLastError();
}

hipError_t launch_sort_edges(uint64_t* keys_a, uint32_t* vals_a, uint64_t* keys_b, uint32_t* vals_b, long long n, int nbits,
                             int low_bits, uint32_t* table, uint32_t* heads, uint32_t* counters, bool* in_b, hipStream_t st) {
    if (in_b) *in_b = false;
    if (n > SORT_MERGE || n <= 0) {
        hipError_t e = launch_radix_sort(keys_a, vals_a, keys_b, vals_b, n, nbits, low_bits, table, in_b, st);
        if (e != hipSuccess) return e;
    } else {
        int passes = 0;
        const int chunk = n > (1 << 18) ? 2 * SORT_CHUNK : SORT_CHUNK;
        if (n > SORT_ONE)
            for (long long run = chunk; run < n; run *= 8) passes++;
        // the last pass writes to keys_a
        uint64_t *ki = keys_a, *ko = passes & 1 ? keys_b : keys_a;
        uint32_t *vi = vals_a, *vo = passes & 1 ? vals_b : vals_a;
        const bool list = passes == 0 && heads;
        uint32_t *lh = list ? heads : nullptr, *lc = list ? counters : nullptr;
        hipError_t ec;
        if (passes > 0 ? chunk == SORT_CHUNK : n > 1024 && n <= 2048) ec = launch_sort_chunk<512, SORT_CHUNK / 512>(ki, vi, ko, vo, n, lh, lc, st);
        else if (n <= 64) ec = launch_sort_chunk<64, 1>(ki, vi, ko, vo, n, lh, lc, st);
        else if (n <= 256) ec = launch_sort_chunk<64, 4>(ki, vi, ko, vo, n, lh, lc, st);
        else if (n <= 1024) ec = launch_sort_chunk<256, 4>(ki, vi, ko, vo, n, lh, lc, st);
        else ec = launch_sort_chunk<1024, 4>(ki, vi, ko, vo, n, lh, lc, st);
        if (ec != hipSuccess || list) return ec;
        for (long long run = chunk; passes > 0; passes--, run *= 8) {
            ki = ko;
            vi = vo;
            ko = ki == keys_a ? keys_b : keys_a;
            vo = vi == vals_a ? vals_b : vals_a;
            const dim3 grid((unsigned)((n + 255) / 256));
            if (n <= 2 * run)
                hipLaunchKernelGGL(merge_runs_kernel<2>, grid, dim3(256), 0, st, ki, vi, ko, vo, (int)n, (int)run);
            else if (n <= 4 * run)
                hipLaunchKernelGGL(merge_runs_kernel<4>, grid, dim3(256), 0, st, ki, vi, ko, vo, (int)n, (int)run);
            else
                hipLaunchKernelGGL(merge_runs_kernel<8>, grid, dim3(256), 0, st, ki, vi, ko, vo, (int)n, (int)run);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!heads) return hipSuccess;
    hipError_t e = launch_fill_u32(counters, 16, 0u, st);
    if (e != hipSuccess) return e;
    return launch_segment_heads(in_b && *in_b ? keys_b : keys_a, n, heads, counters, st);
}

hipError_t launch_scan_u32(uint32_t* data, long long n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(radix_scan_kernel, dim3(1), dim3(1024), 0, st, data, n);
    return hipGetLastError();
}

hipError_t launch_argmin(const double* dist, long long n, uint32_t* out_id, hipStream_t st) {
    hipLaunchKernelGGL(argmin_kernel, dim3(1), dim3(1024), 0, st, dist, n, out_id);
    return hipGetLastError();
}

hipError_t launch_segment_heads(const uint64_t* keys, long long n, uint32_t* heads, uint32_t* nseg, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(segment_heads_kernel, dim3((unsigned)((n + 4095) / 4096)), dim3(1024), 0, st, keys, n, heads, nseg);
    return hipGetLastError();
}

}  // namespace jx
