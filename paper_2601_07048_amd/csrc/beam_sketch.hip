// beamSearch of float32 vectors through byte copies ("sketches") of them.
//
// A search evaluates some thirty neighbours per expansion, and late in it three or four of them enter the frontier: of 3,967
// evaluations of a d = 960 search at L = 128 on 20,000 points 293 do, and 158 more come before the frontier is full.  The
// others have to be shown to be farther than the worst entry, for which a quarter of the bytes will do: next to each vector
// x stands a record x' = m + s c with 8-bit codes c and e >= |x - x'|.  From |q - x| >= |q' - x'| - e - eq a neighbour whose
// bound lies above the worst entry's distance cannot enter (a frontier changes by keys below the worst one only), and is
// left out; the rest, 503 of 3,967 above, is evaluated on the vectors by eval_batch as in beam_search_kernel.  Frontier
// sequence, results, expansion lists and number of expansions are that kernel's, bit for bit, whatever the codes are worth: a
// loose bound costs evaluations, never an entry.  The number of neighbours looked at is not above 256 dimensions: the visited
// table is smaller there (launch_sketch_shape) and forgets more of them.
//
// Bound: the gather.  Why matrix instructions: the query stands as 16-bit integers v = 256 h + l in rows of operand A (h
// and l in turn, so that every lane group receives both sums), 16 neighbours' codes are operand B as they are loaded, and
// <c, h>, <c, l> are exact integers: no conversion, no reduction, one instruction per 1 KB of codes, where the float form
// takes eight vector instructions per chunk and six reduction steps per neighbour.
// Measured: search of a 20,000 x 960 build 31.3 -> 15.7 ms; 30,000 x 960, 2,500 queries, L = 16 / 64 / 128 / 200 852 / 1,658 /
// 2,984 / 5,000 -> 336 / 727 / 1,105 / 2,185 us; 15,000 x 1536 1,567 / 4,331 / 7,133 / 9,539 -> 580 / 1,379 / 2,458 / 4,076.
#include <stdio.h>
#include "beam_kernels.h"

namespace jx {

typedef int v4i __attribute__((ext_vector_type(4)));

// Roundings of the bound.  With X = |x'| + 2 |m| sqrt(d) and Y = |q'|, every sum below errs by less than 4e-6 (X^2 + Y^2)
// (36 float32 roundings of the largest sums, 2^-24 each, and a few of their products); the record carries |x'|^2 - 8e-6 X^2
// and the query |q'|^2 - 8e-6 Y^2.  SKETCH_REL covers the roundings of the float32 distance itself (24 + 6 + 3 of them, all
// terms positive) and of the bound's last steps, SKETCH_ABS subnormal squares.
#define SKETCH_SLACK 8e-6f
#define SKETCH_REL 2e-5f
#define SKETCH_ABS 1e-30f
// coordinates beyond this have no sketch: squares of 1,536 of them stay finite
#define SKETCH_MAX 1e17f
#define SKETCH_DIM 1536  // most dimensions (jx_create: vectors of at most 6,144 bytes)

// record: codes (d bytes, zeros up to a multiple of 16), then {|x'|^2 - slack, m, s, e}
// One wavefront per vector; e = inf where the vector has no sketch (then the bound never holds).
__global__ void __launch_bounds__(256) sketch_kernel(const float* x, long long n, int d, uint8_t* sk, int stride) {
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int lane = lane_id();
    const float* v = x + (size_t)i * d;
    const int nch = (d + 15) / 16;
    uint8_t* rec = sk + (size_t)i * stride;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    bool ok = true;
    for (int c = lane; c < d / 4; c += 64) {
        const float4 w = reinterpret_cast<const float4*>(v)[c];
        const float mx = fmaxf(fmaxf(w.x, w.y), fmaxf(w.z, w.w)), mn = fminf(fminf(w.x, w.y), fminf(w.z, w.w));
        // fmaxf drops a NaN; the sum of absolute values does not
        ok = ok && fabsf(w.x) + fabsf(w.y) + fabsf(w.z) + fabsf(w.w) < 4.f * SKETCH_MAX;
        hi = fmaxf(hi, mx);
        lo = fminf(lo, mn);
    }
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
        hi = fmaxf(hi, shfl_xor(hi, k));
        lo = fminf(lo, shfl_xor(lo, k));
    }
    ok = ballot(!ok) == 0ull && hi <= SKETCH_MAX && lo >= -SKETCH_MAX;
    const float m = ok ? 0.5f * (lo + hi) : 0.f;
    const float s = ok ? (hi - lo) * (1.f / 255.f) : 0.f;
    const float inv = s > 1e-30f ? 1.f / s : 0.f;  // (a range of no width, or one that no bound will reach: all codes 0)
    float err = 0.f, nn = 0.f;
    for (int c = lane; c < nch * 4; c += 64) {
        uint32_t word = 0;
        if (c < d / 4 && ok) {
            const float4 w = reinterpret_cast<const float4*>(v)[c];
            const float f[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const float code = fminf(fmaxf(rintf((f[k] - m) * inv), -128.f), 127.f);
                const float r = fmaf(-s, code, f[k] - m), y = fmaf(s, code, m);
                err = fmaf(r, r, err);
                nn = fmaf(y, y, nn);
                word |= ((uint32_t)(int)code & 255u) << (8 * k);
            }
        }
        reinterpret_cast<uint32_t*>(rec)[c] = word;
    }
    err = group_sum<64>(err);
    nn = group_sum<64>(nn);
    if (lane == 0) {
        const float X = sqrtf(nn) + 2.f * fabsf(m) * sqrtf((float)d);
        // the residuals carry a rounding of f - m (2^-24 of 128 s at most) each, their sum some thirty
        const float e = sqrtf(err) * 1.001f + s * 2e-5f * sqrtf((float)d) + 1e-20f;
        float4 meta = make_float4(nn - SKETCH_SLACK * X * X, m, s, ok ? e : __builtin_inff());
        *reinterpret_cast<float4*>(rec + (size_t)nch * 16) = meta;
    }
}

hipError_t launch_sketch(const float* x, long long n, int d, uint8_t* sk, int stride, hipStream_t st) {
    const long long most = 1 << 24;  // a launch has fewer than 2^32 threads
    for (long long i = 0; i < n; i += most) {
        const long long m = n - i < most ? n - i : most;
        hipLaunchKernelGGL(sketch_kernel, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, st, x + (size_t)i * d, m, d, sk + (size_t)i * stride, stride);
    }
    return hipGetLastError();
}

// Whether copies say something about a set: of up to 256 of its vectors, how many have an uncertainty of their bound, 2 e D +
// 2 slack, of more than a tenth of D^2, D the distance to the next of them (counts[0]; pairs of copies are not counted in
// counts[1]).  Sets far from the origin or of few large coordinates have: every neighbour is kept then, and a query that
// tries 256 of them first is 2 to 20 % slower than without copies, 25 to 50 % with six chunks per lane.  Measured median / times
// as fast as without, L = 64, 2,000 queries of d = 960: Gaussian mixtures of unit deviation moved by 0 / 30 / 100 / 300 0.01 / 2.6,
// 0.04 / 2.4, 0.26 / 0.94, 2.5 / 0.95, with an offset per coordinate of deviation 3 / 30 / 300 0.02 / 2.5, 0.20 / 0.95, 2.4 / 0.94;
// norms over three decades 0.01 / 1.3, fifth powers of normal values 0.03 / 1.5
// One wavefront per vector; x may be of any alignment.
__global__ void __launch_bounds__(256) sketch_probe_kernel(const float* x, long long n, int d, uint32_t* counts) {
    const int lane = lane_id();
    const long long some = n < 256 ? n : 256, w = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= some) return;
    const float *v = x + (size_t)(w * n / some) * d, *o = x + (size_t)((w + 1) % some * n / some) * d;
    float a[SKETCH_DIM / 64], b[SKETCH_DIM / 64];  // all loads in flight at once
#pragma unroll
    for (int k = 0; k < SKETCH_DIM / 64; k++) {
        const int c = k * 64 + lane;
        a[k] = c < d ? v[c] : 0.f;
        b[k] = c < d ? o[c] : 0.f;
    }
    float lo = __builtin_inff(), hi = -__builtin_inff();
    bool ok = true;
#pragma unroll
    for (int k = 0; k < SKETCH_DIM / 64; k++) {
        ok = ok && fabsf(a[k]) <= SKETCH_MAX && fabsf(b[k]) <= SKETCH_MAX;
        hi = fmaxf(hi, k * 64 + lane < d ? a[k] : hi);
        lo = fminf(lo, k * 64 + lane < d ? a[k] : lo);
    }
    ok = ballot(!ok) == 0ull;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
        hi = fmaxf(hi, shfl_xor(hi, k));
        lo = fminf(lo, shfl_xor(lo, k));
    }
    const float m = 0.5f * (lo + hi), s = (hi - lo) * (1.f / 255.f), inv = s > 1e-30f ? 1.f / s : 0.f;
    float err = 0.f, nn = 0.f, dd = 0.f;
#pragma unroll
    for (int k = 0; k < SKETCH_DIM / 64; k++)
        if (k * 64 + lane < d) {
            const float code = fminf(fmaxf(rintf((a[k] - m) * inv), -128.f), 127.f);
            const float r = fmaf(-s, code, a[k] - m), y = fmaf(s, code, m), t = a[k] - b[k];
            err = fmaf(r, r, err);
            nn = fmaf(y, y, nn);
            dd = fmaf(t, t, dd);
        }
    err = group_sum<64>(err);
    nn = group_sum<64>(nn);
    dd = group_sum<64>(dd);
    const float X = sqrtf(nn) + 2.f * fabsf(m) * sqrtf((float)d);
    const bool poor = !ok || 2.f * sqrtf(err * dd) + 2.f * SKETCH_SLACK * X * X > 0.1f * dd;
    if (lane == 0 && (!ok || dd > 0.f)) {
        atomicAdd(&counts[1], 1u);
        if (poor) atomicAdd(&counts[0], 1u);
    }
}

hipError_t launch_sketch_probe(const float* x, long long n, int d, uint32_t* counts, hipStream_t st) {
    if (n >= 2) hipLaunchKernelGGL(sketch_probe_kernel, dim3(64), dim3(256), 0, st, x, n, d, counts);
    return hipGetLastError();
}

// <c, l> and <c, h> of neighbours first + 16 p .. (p < NP) in the lanes of their numbers; KU loads of each in flight.
// lq(k): this lane's part of operand A (rows l, h, l, h, ...; columns 64 k + 16 (lane / 16) ..).  Where d is no multiple of 64 a lane
// group reads up to 48 bytes behind the codes: the rest of the record, whose stride is a multiple of 64 that holds the codes and the
// 16 bytes of their scale.  The query is zero there.
template <int NP, int KU, typename Operand>
__device__ __forceinline__ void sketch_dots(const uint8_t* sk, const uint32_t stride, const int kb, const Operand& lq,
                                            const uint32_t* cand_id, const int first, const int n, const int lane, int& il, int& ih) {
    const uint8_t* rec[NP];
    v4i acc[NP];
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const int c = first + p * 16 + (lane & 15);
        rec[p] = sk + (size_t)cand_id[c < n ? c : n - 1] * stride + (lane >> 4) * 16;
        acc[p] = v4i{0, 0, 0, 0};
    }
    for (int k0 = 0; k0 < (KU == 4 ? 4 : kb); k0 += KU) {  // (KU = 4: kb <= 4)
        v4i b[NP][KU];
#pragma unroll
        for (int p = 0; p < NP; p++)
            if (first + p * 16 < n) {
#pragma unroll
                for (int u = 0; u < KU; u++)
                    if (k0 + u < kb) b[p][u] = *reinterpret_cast<const v4i*>(rec[p] + (size_t)(k0 + u) * 64);
            }
#pragma unroll
        for (int u = 0; u < KU; u++)
            if (k0 + u < kb) {
                const v4i aq = lq(k0 + u);
#pragma unroll
                for (int p = 0; p < NP; p++)
                    if (first + p * 16 < n) acc[p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aq, b[p][u], acc[p], 0, 0, 0);
            }
    }
#pragma unroll
    for (int p = 0; p < NP; p++)
        if ((lane >> 4) * 16 == first + p * 16) {
            il = acc[p][0];
            ih = acc[p][1];
        }
}

// The same with four neighbouring lanes on a record: a quarter of the wavefront then touches 4 lines of a load and not 16, which
// is what the address unit counts, at the price of eight dot products by the vector unit for each.  For batches that fill the
// card (sketch_dots / this, 20,000 x 960 built 27.5 / 27.1 ms, 2,600 queries of d = 960, L = 16 / 128 348 / 335, 1,184 / 1,134 us);
// a lone wavefront waits for those instructions (513 queries 410 / 426, d = 1536 1,011 / 1,053 at L = 64 and 128).
template <int NP, int KU>
__device__ __forceinline__ void sketch_dots_rows(const uint8_t* sk, const uint32_t stride, const int kb, const uint8_t* qpl, const int plane,
                                                 const uint32_t* cand_id, const int first, const int n, const int lane, int& il, int& ih) {
    const uint8_t* rec[NP];
    int lo[NP], hi[NP];
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const int c = first + p * 16 + (lane >> 2);
        rec[p] = sk + (size_t)cand_id[c < n ? c : n - 1] * stride + (lane & 3) * 16;
        lo[p] = hi[p] = 0;
    }
    const uint8_t* ql = qpl + (lane & 3) * 16;
    for (int k0 = 0; k0 < kb; k0 += KU) {
        v4i b[NP][KU];
#pragma unroll
        for (int p = 0; p < NP; p++)
            if (first + p * 16 < n) {
#pragma unroll
                for (int u = 0; u < KU; u++)
                    if (k0 + u < kb) b[p][u] = *reinterpret_cast<const v4i*>(rec[p] + (size_t)(k0 + u) * 64);
            }
#pragma unroll
        for (int u = 0; u < KU; u++)
            if (k0 + u < kb) {
                const v4i vl = *reinterpret_cast<const v4i*>(ql + (size_t)(k0 + u) * 64);
                const v4i vh = *reinterpret_cast<const v4i*>(ql + plane + (size_t)(k0 + u) * 64);
#pragma unroll
                for (int p = 0; p < NP; p++)
                    if (first + p * 16 < n) {
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            lo[p] = __builtin_amdgcn_sdot4(b[p][u][e], vl[e], lo[p], false);
                            hi[p] = __builtin_amdgcn_sdot4(b[p][u][e], vh[e], hi[p], false);
                        }
                    }
            }
    }
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const int x = __builtin_amdgcn_ds_bpermute((lane & 15) * 16, group_sum<4>(lo[p]));
        const int y = __builtin_amdgcn_ds_bpermute((lane & 15) * 16, group_sum<4>(hi[p]));
        if ((lane >> 4) * 16 == first + p * 16) {
            il = x;
            ih = y;
        }
    }
}

// bytes of one query plane in LDS (a bank group apart from the other)
__host__ __device__ inline int sketch_plane(int nch_codes) { return (nch_codes + 3) / 4 * 64 + 16; }

// The query in 16 bits, q' = scale v with |q - q'| <= err, its planes l and h in LDS; none: it has no such form.
struct SketchQuery {
    float scale, err, norm, sum;  // norm: |q'|^2 less the slack; sum: of the coordinates of q'
    bool none;
};

// By a whole wavefront; rec: nch chunks of four floats
__device__ __forceinline__ SketchQuery sketch_query(const uint8_t* rec, const int nch, const int kb, uint8_t* qpl, const int plane, const int lane) {
    SketchQuery o;
    const float4* qv = reinterpret_cast<const float4*>(rec);
    float mx = 0.f;
    bool ok = true;
    for (int c = lane; c < nch; c += 64) {
        const float4 w = qv[c];
        ok = ok && fabsf(w.x) + fabsf(w.y) + fabsf(w.z) + fabsf(w.w) < 4.f * SKETCH_MAX;  // false for a NaN
        mx = fmaxf(mx, fmaxf(fmaxf(fabsf(w.x), fabsf(w.y)), fmaxf(fabsf(w.z), fabsf(w.w))));
    }
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) mx = fmaxf(mx, shfl_xor(mx, k));
    o.none = ballot(!ok) != 0ull || !(mx <= SKETCH_MAX);
    o.scale = mx * (1.f / 32639.f);
    const float inv = o.scale > 1e-30f ? 1.f / o.scale : 0.f;
    float err = 0.f, nn = 0.f;
    int vsum = 0;
    for (int c = lane; c < kb * 16; c += 64) {
        uint32_t wl = 0, wh = 0;
        if (c < nch && !o.none) {
            const float4 w = qv[c];
            const float f[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const float code = fminf(fmaxf(rintf(f[k] * inv), -32639.f), 32639.f);
                const float r = fmaf(-o.scale, code, f[k]), y = o.scale * code;
                err = fmaf(r, r, err);
                nn = fmaf(y, y, nn);
                const int v = (int)code, h = (v + 128) >> 8;  // v = 256 h + l, both in [-128, 127]
                vsum += v;
                wh |= ((uint32_t)h & 255u) << (8 * k);
                wl |= ((uint32_t)(v - 256 * h) & 255u) << (8 * k);
            }
        }
        reinterpret_cast<uint32_t*>(qpl)[c] = wl;
        reinterpret_cast<uint32_t*>(qpl + plane)[c] = wh;
    }
    err = group_sum<64>(err);
    nn = group_sum<64>(nn);
    vsum = group_sum<64>(vsum);
    o.err = sqrtf(err) * 1.001f + 1e-20f;
    o.norm = nn - SKETCH_SLACK * nn;
    o.sum = o.scale * (float)vsum;
    return o;
}

// |q' - x'|^2 less the slack of both, from the two sums of sketch_dots and the record's meta chunk
__device__ __forceinline__ float sketch_dist(const SketchQuery& q, const float4 meta, const int il, const int ih) {
    const float dot = fmaf(256.f, (float)ih, (float)il);
    const float t = fmaf(meta.z * dot, q.scale, meta.y * q.sum);  // <x', q'>
    return fmaf(-2.f, t, meta.x + q.norm);
}

// Copies take a round trip of their own before the vectors'.  Where an expansion has few new neighbours, whose vectors come in one
// round trip, they only make it longer: norms over three decades (some five new neighbours per expansion), without copies /
// copies of all / of more than these, 60,000 x 132, L = 64, 2,000 queries 253 / 300 / 255 us, 20,000 x 512, L = 256 803 / 938 /
// 805, 20,000 x 960, 16 calls of 32 points 10,297 / 10,573 / 9,414; 5,000 x 1536, L = 128, 4,000 queries of fifth powers of normal
// values 712 / 901 / 603.  With 8 instead of 4 a build of 20,000 x 960 took 27.9 for 27.7 ms
template <int T, int CPL, int KU>
constexpr int sketch_few() { return T * CPL <= 64 || (CPL == 6 && KU == 16) ? 8 : 4; }

// Tag table and rows of at most 64 entries only (the launcher checks).  KU: 64-byte pieces of two tiles of 16 neighbours in
// flight, as the registers allow for four wavefronts per SIMD (codes of at most 256 bytes: KU = 4; 40,000 x 200 built with
// KU = 4 / five wavefronts, spilled / four tiles 16.2 / 18.5 / 16.6 ms), three (8) or two (16: batches that fill no more).
template <int T, int CPL, int NREG, bool VIS, int KU>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(KU == 4 ? 4 : (KU == 8 ? 3 : 2), 8))) beam_search_sketch_kernel(BeamArgs a) {
    constexpr int G = 64 / T;
    constexpr int U0 = CPL == 4 ? 4 : (CPL == 6 ? 2 : 8 / CPL);  // (one of six chunks: 30,000 x 1536, L = 10, 600 queries 251 -> 188 us)
    constexpr int U = U0 < (64 / G) ? U0 : (64 / G);
    constexpr int FCAP = mirror_entries<NREG>();
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int g = lane / T, lig = lane % T;
    const int64_t qi = blockIdx.x;
    if (qi >= a.nq) return;

    const int tag_bits = a.tag_bits;
    const uint32_t id_mask = (1u << (tag_bits + 30 - __builtin_clz((uint32_t)a.hash_slots))) - 1u;  // hash_slots / 2 sets
    const int plane = sketch_plane(a.sk_nch), kb = (a.sk_nch + 3) / 4;
    constexpr bool HELD = KU == 4;  // the query's planes in 16 registers; they stand in the table's room until they are read
    uint64_t* fr = reinterpret_cast<uint64_t*>(smem + (HELD ? 0 : 2 * plane));
    uint64_t* cand_key = fr + FCAP;
    uint32_t* cand_id = reinterpret_cast<uint32_t*>(cand_key + 64);
    uint32_t* tab = cand_id + 64;
    uint8_t* const qpl = HELD ? reinterpret_cast<uint8_t*>(tab) : smem;
    const auto clear = [=]() __attribute__((always_inline)) {
        for (int i = lane; i < a.hash_slots / 2; i += 64) tab[i] = JX_NONE_ID;
        for (int i = lane; i < FCAP; i += 64) fr[i] = JX_EMPTY_KEY;
    };
    if constexpr (!HELD) clear();

    const int64_t qrec = qi + (qi >= a.q_skip ? 1 : 0);
    QueryRegs<K_F32, CPL, 0> q;
    load_query<K_F32, T, CPL, 0>(q, a.ds, qrec, lig);

    const SketchQuery sq = sketch_query(a.ds.qrecs + qrec * a.ds.qrec_stride, a.ds.nch, kb, qpl, plane, lane);
    bool use = !sq.none;
    const uint8_t* my_q = qpl + (lane & 1) * plane + (lane >> 4) * 16;
    v4i held[4];
    if constexpr (HELD) {
        wave_sync();
#pragma unroll
        for (int k = 0; k < 4; k++) held[k] = k < kb ? *reinterpret_cast<const v4i*>(my_q + k * 64) : v4i{0, 0, 0, 0};
        wave_sync();
        clear();
        wave_sync();
    }
    const auto lq = [&](const int k) __attribute__((always_inline)) {
        if constexpr (HELD) return held[k];
        else return *reinterpret_cast<const v4i*>(my_q + (size_t)k * 64);
    };

    uint64_t fk[NREG];
#pragma unroll
    for (int r = 0; r < NREG; r++) fk[r] = JX_EMPTY_KEY;
    int count = 0;
    uint64_t worst = JX_EMPTY_KEY;  // see frontier_merge
    const int L = a.L;
    const bool full = a.ds.nch == T * CPL;
    uint32_t hops = 0, evals = 0;
    uint64_t vk = 0;  // VIS: see visited_add
    int tried = 0, kept = 0;  // by sketches: copies read, vectors read after them

    if (lane == 0) {  // seed: the entry vertex
        cand_id[0] = a.entry;
        const uint32_t h = (a.entry * 0x9E3779B1u) & id_mask;
        tab[h >> tag_bits] = 0xFFFF0000u | (h & ((1u << tag_bits) - 1u));
    }
    wave_sync();
    eval_batch<K_F32, T, CPL, 0, 1>(q, a.ds, 0, 1, cand_id, cand_key, g, lig);
    wave_sync();
    if (lane == 0) {
        fk[0] = cand_key[0];
        fr[0] = cand_key[0];
    }
    wave_sync();
    count = 1;
    evals = 1;

    // the loop of beam_search_body's MODE 1, with step 4a
    const uint32_t* my_adj = a.adj + (lane < a.R ? lane : 0);
    uint32_t row_u = a.entry, row_v = my_adj[(size_t)a.entry * (uint32_t)a.R];
    for (;;) {
        // ---- 1. the two closest unexpanded entries
        uint64_t ukey = 0;
        uint32_t u2 = 0;
        int sel_r = -1, sel_lane = 0;
        bool have2 = false;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            uint64_t m = ballot((fk[r] & 1ull) == 0ull);
            if (sel_r < 0 && m != 0ull) {
                sel_r = r;
                sel_lane = __builtin_ctzll(m);
                ukey = readlane64(fk[r], sel_lane);
                m &= m - 1ull;
            }
            if (!have2 && m != 0ull) {
                have2 = true;
                u2 = readlane32((uint32_t)fk[r], __builtin_ctzll(m)) >> 1;
            }
        }
        if (sel_r < 0) break;
        const uint32_t u = key_id(ukey);
#pragma unroll
        for (int r = 0; r < NREG; r++) fk[r] |= (r == sel_r && lane == sel_lane) ? 1ull : 0ull;
        if constexpr (VIS) {
            visited_add(a, qi, vk, hops, ukey | 1ull, lane);
        }
        hops++;
        // ---- 2. adjacency row
        if (row_u != u) row_v = my_adj[(size_t)u * (uint32_t)a.R];
        const uint32_t v = lane < a.R ? row_v : JX_NONE_ID;
        // ---- 3. visited filter
        const uint32_t h = (v * 0x9E3779B1u) & id_mask;
        const uint32_t tag = h & ((1u << tag_bits) - 1u);
        const uint32_t w = tab[h >> tag_bits];
        row_u = have2 ? u2 : u;
        row_v = my_adj[(size_t)row_u * (uint32_t)a.R];
        const bool is_new = v != JX_NONE_ID && (w & 0xFFFFu) != tag && (w >> 16) != tag;
        const uint64_t nm = ballot(is_new);
        if (nm == 0ull) continue;
        int n_new = __builtin_popcountll(nm);
        if (is_new) {
            tab[h >> tag_bits] = (w << 16) | tag;
            cand_id[prefix_count(nm)] = v;
        }
        wave_sync();
        evals += n_new;
        // ---- 4a. which of them may enter a full frontier
        if (use && worst != JX_EMPTY_KEY && n_new > sketch_few<T, CPL, KU>()) {
            const uint32_t id = cand_id[lane < n_new ? lane : n_new - 1];
            const float4 meta = *reinterpret_cast<const float4*>(a.sk + (size_t)id * (uint32_t)a.sk_stride + (size_t)a.sk_nch * 16);
            int il = 0, ih = 0;
            for (int f = 0; f < n_new; f += 32) {
                if constexpr (KU == 8)
                    sketch_dots_rows<2, KU>(a.sk, (uint32_t)a.sk_stride, kb, qpl, plane, cand_id, f, n_new, lane, il, ih);
                else
                    sketch_dots<2, KU>(a.sk, (uint32_t)a.sk_stride, kb, lq, cand_id, f, n_new, lane, il, ih);
            }
            const float d2 = sketch_dist(sq, meta, il, ih);
            const float far = sqrtf(ordered_to_f32(key_dist(worst))) + meta.w + sq.err;
            const bool keep = lane < n_new && !(d2 > fmaf(far * far, 1.f + SKETCH_REL, SKETCH_ABS));
            const uint64_t km = ballot(keep);
            const int nk = __builtin_popcountll(km);
            tried += n_new;
            kept += nk;
            // vectors that their codes say little about (far from the origin, say): this query goes on without
            use = kept * 4 <= tried * 3 + 256;
            if (nk == 0) continue;
            if (nk < n_new) {
                wave_sync();
                if (keep) cand_id[prefix_count(km)] = id;
                n_new = nk;
                wave_sync();
            }
        }
        // ---- 4./5. gather + distances
        if (full) {
            for (int s0 = 0; s0 < n_new; s0 += G * U)
                eval_batch<K_F32, T, CPL, 0, U, true>(q, a.ds, s0, n_new, cand_id, cand_key, g, lig);
        } else {
            for (int s0 = 0; s0 < n_new; s0 += G * U)
                eval_batch<K_F32, T, CPL, 0, U, false>(q, a.ds, s0, n_new, cand_id, cand_key, g, lig);
        }
        wave_sync();
        const uint64_t ck = lane < n_new ? cand_key[lane] : JX_EMPTY_KEY;
        wave_sync();
        // ---- 6. merge into the sorted frontier
        frontier_merge<NREG>(fk, fr, count, worst, L, ck, n_new, lane);
    }

    if constexpr (VIS) {
        write_visited<K_F32, NREG>(a, qi, fk, count, worst, vk, reinterpret_cast<uint64_t*>(tab), hops, lane);
        if (a.stats && lane == 0) {
            unsigned long long* sp = a.stats + (size_t)(qi & 63) * 16;
            atomicAdd(&sp[0], (unsigned long long)hops);
            atomicAdd(&sp[1], (unsigned long long)evals);
        }
    } else {
        write_results<K_F32, NREG>(a, qi, fk, count, lane, hops, evals);
        if (a.stats && lane == 0) {
            unsigned long long* sp = a.stats + (size_t)(qi & 63) * 16;
            atomicAdd(&sp[3], (unsigned long long)tried);
            atomicAdd(&sp[4], (unsigned long long)(tried - kept));
        }
    }
}

// ------------------------------------------------------------------ exact re-rank
//
// The first k of at most 64 candidates, by exact distance: as rerank_kernel does it, but what its byte copy shows to be farther
// than k others is not read.  The k-th smallest of the upper bounds (|q' - x'| + e + eq)^2 is no smaller than the k-th distance,
// so a candidate whose lower bound exceeds it is none of the first k.  Bound: the gathers, 40 copies and some twelve vectors of a
// query for 40 vectors.
struct SketchRerankLds {
    uint64_t cand_key[64];
    uint32_t cand_id[64];
    float bound[64];
};

// MANY: few loads in flight and four to six wavefronts per SIMD (76 to 103 registers), which hold a batch of 4,096 queries; else two
// or three with many (149 to 169).  Whole searches at L = 64 of 4,000 queries on 20,000 vectors, 40 candidates, times as fast as
// with whole vectors in the re-rank, two / four: d = 960 Gaussian mixtures 1.02 / 1.06, normal values 0.91 / 0.99, fifth powers of
// them 0.89 / 0.96, d = 1536 1.07 / 1.09, 0.92 / 0.99, 0.90 / 0.96; 10,000 queries, d = 384 523 / 502, 588 / 551 and 380 / 344 us, d =
// 960 1,195 / 1,185, 1,183 / 1,181 and 652 / 617.  A batch that leaves the card idle waits for its own loads: 64 candidates, 200
// queries of d = 960, normal values 264 / 269 us
template <int T, int CPL, bool MANY>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MANY ? 4 : 2, 8))) rerank_sketch_kernel(RerankArgs a) {
    constexpr int G = 64 / T;
    constexpr int U0 = MANY ? (CPL == 6 ? 2 : 8 / CPL) : (CPL == 2 ? 8 : (CPL == 4 ? 6 : 4));
    constexpr int U = U0 < (64 / G) ? U0 : (64 / G);
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int g = lane / T, lig = lane % T;
    const long long qi = (long long)blockIdx.x * 4 + wave;
    if (qi >= a.nq) return;
    const int plane = sketch_plane(a.sk_nch), kb = (a.sk_nch + 3) / 4;
    unsigned char* my = smem + (size_t)wave * (sizeof(SketchRerankLds) + 2 * (size_t)plane);
    SketchRerankLds* L = reinterpret_cast<SketchRerankLds*>(my);
    uint8_t* qpl = my + sizeof(SketchRerankLds);
    QueryRegs<K_F32, CPL, 0> q;
    load_query<K_F32, T, CPL, 0>(q, a.ds, qi, lig);
    const uint32_t* cand = a.cand + (size_t)qi * a.cand_stride;
    const uint32_t id = lane < a.rr ? cand[lane] : JX_NONE_ID;
    const int m = __builtin_popcountll(ballot(id != JX_NONE_ID));  // the frontier is filled from the left
    if (lane < m) L->cand_id[lane] = id;
    wave_sync();
    int n = m;
    bool use = m > a.k;
    float4 meta = make_float4(0.f, 0.f, 0.f, 0.f);
    if (use) {
        meta = *reinterpret_cast<const float4*>(a.sk + (size_t)L->cand_id[lane < m ? lane : 0] * (uint32_t)a.sk_stride + (size_t)a.sk_nch * 16);
        // Worth it where the estimates put a third of the candidates farther beyond the k-th than both bounds are wide: else most
        // vectors are read after all (a quarter: the same within 0.5 %).  Before MANY, 10,000 queries, without copies / always / a half / a third / a quarter, us: 1M x 1536, 1-bit
        // codes, 40 candidates 400 / 371 / 408 / 390 / 374, 1M x 960, 4 bits 237 / 226 / 228 / 218 / 220; 10,000 x 1536, 64, fifth
        // powers of normal values 141 / 262 / 181 / 193 / 205, a Gaussian mixture 531 / 223 / 224 / 229 / 223
        const float est = lane < m ? a.cand_dist[(size_t)qi * a.cand_stride + lane] : 0.f;
        const float wide = 2.f * sqrtf(fmaxf(est, 0.f)) * meta.w;
        const float bar = __uint_as_float(readlane32(__float_as_uint(est + wide), a.k - 1));
        use = __builtin_popcountll(ballot(lane < m && est - wide > bar)) * 3 >= m;
    }
    SketchQuery sq;
    if (use) {
        sq = sketch_query(a.ds.qrecs + qi * a.ds.qrec_stride, a.ds.nch, kb, qpl, plane, lane);
        use = !sq.none;
        wave_sync();
    }
    if (use) {
        int il = 0, ih = 0;
        const uint8_t* my_q = qpl + (lane & 1) * plane + (lane >> 4) * 16;
        const auto lq = [=](const int k) __attribute__((always_inline)) { return *reinterpret_cast<const v4i*>(my_q + (size_t)k * 64); };
        if (m <= 48) {
            sketch_dots<3, MANY ? 2 : 5>(a.sk, (uint32_t)a.sk_stride, kb, lq, L->cand_id, 0, m, lane, il, ih);
        } else {
            for (int f = 0; f < m; f += 32) sketch_dots<2, MANY ? 3 : 8>(a.sk, (uint32_t)a.sk_stride, kb, lq, L->cand_id, f, m, lane, il, ih);
        }
        const float d2 = sketch_dist(sq, meta, il, ih), off = meta.w + sq.err;
        // upward: the slack twice (it stands below |x'|^2 and |q'|^2, whose sum it is 8e-6 of, X <= |x'| + 2 |m| sqrt(d))
        const float X = sqrtf(fmaxf(meta.x, 0.f)) * 1.001f + 2.f * fabsf(meta.y) * sqrtf((float)(a.sk_nch * 16));
        const float up = sqrtf(fmaxf(d2, 0.f) + 2.02f * SKETCH_SLACK * (X * X + sq.norm * 1.001f)) + off;
        const float most = fmaf(up * up, 1.f + SKETCH_REL, SKETCH_ABS);  // no smaller than the float32 distance
        L->bound[lane] = lane < m && most == most ? most : __builtin_inff();
        wave_sync();
        int rank = 0;
        const float mine = L->bound[lane];
        for (int t = 0; t < m; t++) {
            const float o = L->bound[t];
            rank += o < mine || (o == mine && t < lane) ? 1 : 0;
        }
        const uint64_t kth = ballot(lane < m && rank == a.k - 1);
        const float bar = sqrtf(L->bound[kth ? __builtin_ctzll(kth) : 0]) + off;  // (ranks are distinct: there is one)
        const bool keep = lane < m && !(d2 > fmaf(bar * bar, 1.f + SKETCH_REL, SKETCH_ABS));
        const uint64_t km = ballot(keep);
        n = __builtin_popcountll(km);
        wave_sync();
        if (keep) L->cand_id[prefix_count(km)] = id;
        wave_sync();
    }
    for (int s0 = 0; s0 < n; s0 += G * U) eval_batch<K_F32, T, CPL, 0, U>(q, a.ds, s0, n, L->cand_id, L->cand_key, g, lig);
    wave_sync();
    // rank sort by (distance, id); write the first k, pad what is left
    for (int j = n + lane; j < a.k; j += 64) {
        a.out_ids[qi * a.k + j] = JX_NONE_ID;
        a.out_dist[qi * a.k + j] = __builtin_inff();
    }
    if (lane < n) {
        const uint64_t kj = L->cand_key[lane];
        int rank = 0;
        for (int t = 0; t < n; t++) rank += (L->cand_key[t] < kj) ? 1 : 0;
        if (rank < a.k) {
            a.out_ids[qi * a.k + rank] = key_id(kj);
            a.out_dist[qi * a.k + rank] = ordered_to_f32(key_dist(kj));
        }
    }
    if (a.stats && lane == 0) {
        unsigned long long* sp = a.stats + (size_t)(qi & 63) * 16;
        atomicAdd(&sp[2], (unsigned long long)n);
        if (use) atomicAdd(&sp[5], (unsigned long long)m);
    }
}

hipError_t launch_rerank_sketch(const RerankArgs& a, hipStream_t st, bool* done) {
    *done = false;
    const int nch = a.ds.nch;
    // Whole vectors / this before MANY, us: 41 candidates for 40 neighbours, 10,000 queries 227 / 292; 50,000 x 256, 5,000 queries 33 /
    // 35; Gaussian mixtures of d = 960 / 1536, 64 candidates, 200 queries 42 / 27 and 60 / 38.  Fewer than 2,048 queries with 40
    // candidates lose: 2,100, whole searches with MANY, Gaussian mixtures of d = 384 / 960 / 1536 227 / 225, 459 / 446, 455 / 432, normal
    // values 241 / 245, 394 / 401, 404 / 413, fifth powers 164 / 166, 229 / 237, 264 / 274
    if (!a.sk || a.rr > 64 || a.rr < 3 * a.k || nch <= 64 || nch > 384 || (a.nq < 2048 && a.rr <= 48)) return hipSuccess;
    *done = true;
    const size_t sh = 4 * (sizeof(SketchRerankLds) + 2 * (size_t)sketch_plane(a.sk_nch));
    const dim3 grid((unsigned)((a.nq + 3) / 4));
#define JX_RR(C)                                                                                               \
    if (nch <= 64 * C) {                                                                                       \
        auto kern = a.nq >= 2048 ? rerank_sketch_kernel<64, C, true> : rerank_sketch_kernel<64, C, false>;     \
        hipLaunchKernelGGL(kern, grid, dim3(256), sh, st, a);                                                  \
    }
    JX_RR(2) else JX_RR(4) else JX_RR(6)
#undef JX_RR
    return hipGetLastError();
}

// ------------------------------------------------------------------ launch

template <int T, int CPL>
static hipError_t launch_sketch_shape(BeamArgs a, hipStream_t st, char* name) {
    const int nreg = a.L <= 64 ? 1 : (a.L <= 128 ? 2 : 4);
    constexpr bool SHORT = T * CPL <= 64;
    // two wavefronts per SIMD are 2,048 queries: 15,000 x 1536 at L = 200, 700 / 1,500 / 2,000 queries 1,681 / 2,152 / 3,741 ->
    // 1,505 / 2,046 / 3,478 us, 30,000 x 960 at L = 64 447 / 561 / 649 -> 422 / 541 / 632
    const bool wide = !SHORT && a.sk_nch > 32 && a.nq <= 2048;
    // what the visited table forgets costs a quarter of the bytes here, so a smaller one than the vectors ask for, and more
    // wavefronts by LDS (build of 20,000 x 960, L = 128: 16 / 8 / 4 KB 33.2 / 32.3 / 33.9 ms; 1,500 queries at L = 200 2.19 /
    // 1.99 / 2.19 ms, but 5,000 3.52 / 3.68 / 4.00).  With 16 KB 1,792 queries of more than 128 entries are resident, and the
    // rest of a wide batch waited for them: 2,000 queries on 6,000 x 960, L = 256 1,506 -> 805 us; of fewer none waits, and what the
    // smaller table forgets makes the chain longer (300 queries on 30,000 x 960, L = 256 1,297 / 1,455)
    // Vectors of at most 256 dimensions: 8 KB as without copies; as the planes of the query take no room (HELD), 4,096 queries of 65 to
    // 128 entries are resident, as without copies.  With the planes beside them 3,584 were, or 4 KB for the table: 60,000 x 132, L =
    // 128, 10,000 queries without copies / 4 KB / this 880 / 779 / 746 us, normal data 3,288 / 1,686 / 1,544, 300,000 x 200 1,866 /
    // 1,637 / 1,542 and 6,190 / 2,516 / 2,354; inner products by an extra dimension, where copies say nothing, 1M x 204 3,847 / 4,266 /
    // 3,881
    while (a.hash_slots > (a.L <= 128 || (wide && a.nq > 1792) ? 4096 : 8192) && a.tag_bits < 15) {
        a.hash_slots /= 2;
        a.tag_bits++;
    }
    const size_t sh0 = (SHORT ? 0 : 2 * (size_t)sketch_plane(a.sk_nch)) + 64 * 8 + 64 * 4 + table_bytes(a);
    if (name) snprintf(name, 96, "beam_search_sketch_kernel<%d,%d,%d,%d,%d>", T, CPL, nreg, a.vis_cap ? 1 : 0, SHORT ? 4 : (wide ? 16 : 8));
#define JX_LAUNCH(NR, VISIBLE)                                                                                          \
    {                                                                                                                   \
        const size_t sh = sh0 + mirror_entries<NR>() * 8;                                                               \
        auto kern = SHORT ? beam_search_sketch_kernel<T, CPL, NR, VISIBLE, SHORT ? 4 : 8>                               \
                          : (wide ? beam_search_sketch_kernel<T, CPL, NR, VISIBLE, SHORT ? 4 : 16>                      \
                                  : beam_search_sketch_kernel<T, CPL, NR, VISIBLE, SHORT ? 4 : 8>);                     \
        hipLaunchKernelGGL(kern, dim3((unsigned)a.nq), dim3(64), sh, st, a);                                            \
        return hipGetLastError();                                                                                       \
    }
    if (a.vis_cap) {
        if constexpr (SHORT || CPL == 2) {
            return hipErrorInvalidValue;  // no expansion lists of such vectors (visited_list_offered)
        } else {
            if (nreg == 1) JX_LAUNCH(1, true)
            JX_LAUNCH(2, true)
        }
    }
    if (nreg == 1) JX_LAUNCH(1, false)
    if (nreg == 2) JX_LAUNCH(2, false)
    if constexpr (!SHORT) JX_LAUNCH(4, false)
    return hipErrorInvalidValue;
#undef JX_LAUNCH
}

hipError_t launch_beam_sketch(int kind, const BeamArgs& a, hipStream_t st, char* name, bool* done) {
    *done = false;
    const int nch = a.ds.nch;
    // Switches that change nothing about these searches; with any other one whole vectors are read.  Batches that a team of
    // wavefronts per query serves without a switch (launch_beam_ahead): with one they run on the one-wavefront kernel, whose
    // visited table and counters are the team's.  A search for expansion lists has no other forms; a table of another kind has
    // no tag_bits
    uint32_t indifferent = JX_FLAG_NO_INCR_PRUNE | JX_FLAG_NO_GRAM | JX_FLAG_GRAM_U8;
    if (a.nq > 512) indifferent |= JX_FLAG_NO_PAIR | JX_FLAG_LANES_NARROW | (nch > 64 ? JX_FLAG_LANES_WIDE : 0u);
    if (a.vis_cap) indifferent = JX_FLAG_ALL;
    if (kind != K_F32 || !a.sk || a.tag_bits == 0 || a.R > 64 || a.L > 256 || (a.flags & ~indifferent)) return hipSuccess;
    if (a.vis_cap && (a.L > 128 || nch <= 128)) return hipSuccess;
    // short vectors and wide frontiers: 60,000 x 200 at L = 128 / 200, 1,000 queries 439 / 596 -> 405 / 588 us, 3,500 473 / 701 ->
    // 429 / 863
    *done = true;
    if (nch <= 64 && a.L <= 128) return launch_sketch_shape<32, 2>(a, st, name);
    if (nch > 64 && nch <= 128) return launch_sketch_shape<64, 2>(a, st, name);
    if (nch > 128 && nch <= 256) return launch_sketch_shape<64, 4>(a, st, name);
    if (nch > 256 && nch <= 384) return launch_sketch_shape<64, 6>(a, st, name);
    *done = false;
    return hipSuccess;
}

}  // namespace jx
