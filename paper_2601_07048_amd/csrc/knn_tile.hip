// Exhaustive k-nearest-neighbour search on the matrix cores.
//
// A 256-thread workgroup owns 128 queries and streams a slice of the base set in steps of 128 vectors.  Each of its
// four wavefronts computes a 64 x 64 block of <q, b> (32x32 MFMA tiles, operands staged through LDS in slabs of 128
// bytes a row, the next slab on its way in registers), and d = |q|^2 + |b|^2 - 2 <q, b> is compared with the query's
// threshold, one add and one compare per pair.  What passes is appended to a 32-entry buffer of the query in LDS; a
// buffer that is nearly full is merged into the query's sorted list of this slice (global memory, L2) by one wavefront,
// which also renews the threshold: every slice publishes a few of its smallest distances, and enough of all slices'
// published ones bound the k-th of all (knn_limit), so a slice accepts little that the whole set would not accept.
//
//   uint8            v_mfma_i32_32x32x32_i8 on the values shifted by -128 (distances do not change): exact integers, so
//                    the lists hold the result.
//   float32/binary16 v_mfma_f32_32x32x16_bf16 on two bfloat16 parts of each value (three products: 96 cycles for 16
//                    coordinates, 512 by 32x32x2_f32; three parts up to 16 dimensions) / 32x32x16_f16: these distances only
//                    choose KNN_SLACK more candidates than asked for.  The merge kernel evaluates them with the arithmetic of bruteforce_tile_kernel,
//                    operation by operation, orders them, and proves that nothing left out can be among the first
//                    k: the first distance left out, less the error bound of both forms (knn_bound.h), has to exceed
//                    the k-th one.
//                    Queries for which it does not (ties, sets far from the origin) are flagged, and their tiles are done
//                    again by bruteforce_tile_kernel.  So the result is that kernel's, bit for bit.
//
// Bound: float32 staging and barriers, a slab in 1.85 us where its products take 0.64 (0.68 of the 1.1 ms below; 1.8 ms on the
// float32 instruction), uint8 likewise (2.0 of 2.75 ms), then appends and merges.  Against bruteforce_tile_kernel:
// 10,000 x 1M uint8 d = 128, k = 10 27.2 -> 2.72 ms; 1,000 x 100,003 float32 d = 960, k = 100 13.0 -> 1.16 ms; 1,000 x 100,000
// binary16 d = 960, k = 10 3.97 -> 0.58 ms; 100 x 1M uint8 d = 128, k = 10 0.076 ms.  Without the seeds the lists fill with
// what comes first: 5.6 and 5.3 ms before these forms.
#include <stdio.h>
#include "jx_distance.h"
#include "knn_bound.h"

namespace jx {

typedef float kf32x16 __attribute__((ext_vector_type(16)));
typedef int ki32x16 __attribute__((ext_vector_type(16)));
typedef int ki32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 kf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 kbf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 kbf16x2 __attribute__((ext_vector_type(2)));
typedef float kf32x2 __attribute__((ext_vector_type(2)));

#define KROW 144      // bytes of a staged row: 128 and 16 of padding
#define KCAP 32       // buffer entries per query
#define KFLUSH 28     // a buffer with this many entries is merged: with 16, 24, 28 1,000 x 300,000 uint8 d = 96, k = 100 1,153, 966, 852 us
#define KU8_ROW 16384    // uint8: longest row, see KINF
// uint8: above every distance (16,384 x 255^2 is just under 2^30), and no sum overflows: 2 <q, b> of the shifted values is at most
// 2^29, |q|^2 at most 2^28, so 2 <q, b> + KINF - |q|^2 stays below 2^31 and 2 <q, b> - |b|^2 above -2^30
#define KINF 0x50000000

#define KNN_SLACK 28  // float types: candidates kept beyond k
#define KNN_BLOCKS 512   // and so the largest number of slices
#define KNN_ENTRIES 512  // published distances of a query, all slices (KNN_PUB of one)
#define KNN_ODD 30  // rows that are listed for the merge of a query tile, see KnnOdd

// Rows of the base set that no threshold can decide on: float32 with a NaN, binary16 with a NaN or an infinity.  They are kept
// out of the lists, and the merge evaluates them for every query; more than KNN_ODD of them leave its results unproven.
struct KnnOdd {
    uint32_t count;
    uint32_t bb_max;  // largest |b|^2 of the other rows (float bits)
    uint32_t id[KNN_ODD];
};

template <int DT>
constexpr uint32_t KNN_DECIDABLE = DT == JX_F16 ? 0x7F800000u : 0x7F800001u;  // bits of |b|^2 from which a row is one of those

struct KnnArgs {
    const void* base;
    const void* queries;
    long long n, nq;
    int d, nch;         // dimensions, 16-byte chunks per vector
    int k, kp;          // neighbours asked for, kept per list
    float parts;        // knn_parts of float32, else 0
    int nsplit;
    uint64_t* lists;    // [nq][nsplit][kp] keys (distance, id)
    uint32_t* published;  // [nq][nsplit][pub] distances of each slice's entries 2^pub_shift - 1, 2 2^pub_shift - 1, .., or NULL
    int r_th;           // ceil(kp / nsplit)
    int pub, pub_shift;
    int seed_steps;     // > 0: the slices' first thresholds come from their first seed_steps steps
    uint32_t* redo;     // [nq] the first limits, then (float types) 1 = the merge could not prove the result
    KnnOdd* odd;        // [tiles of KT queries] float types
    uint4* hopeless;    // [tiles][nsplit] float types: a bit per query that can hardly be proven, as far as the slice can tell
    uint32_t* out_ids;
    float* out_dist;
};

template <int DT> struct KAcc { typedef kf32x16 type; typedef float elem; };
template <> struct KAcc<JX_U8> { typedef ki32x16 type; typedef int elem; };

// The query tile (.x) and slice (.y) of a workgroup.  Workgroups go round the eight XCDs by their number; consecutive tiles of
// one slice are given to one XCD, whose workgroups then stream the same vectors through its L2.  In order of their numbers /
// like this, k = 10: 1,000 x 200,000 float32 d = 128 416 / 372 us, 1,000 x 100,000 d = 960 1,022 / 986, 300 x 50,000 d = 1536 455 /
// 441, binary16 1,000 x 100,000 d = 960 531 / 520.  uint8 above 128 bytes: 1,000 x 100,000 d = 144 134.6 / 132.6, d = 256 136.7 /
// 138.5, 300 x 300,000 d = 256 133.3 / 131.7, d = 960 271 / 259, 10,000 x 200,000 d = 256 1,588 / 1,581, d = 960 4,240 / 4,147.
// Not knn_u8_kernel: 5,000 x 300,000 d = 96, k = 100 1,774 / 1,808.
__device__ __forceinline__ int2 knn_work(const KnnArgs& a) {
    const uint32_t g = gridDim.x, xcd = blockIdx.x & 7u, each = g >> 3, more = g & 7u;
    const uint32_t w = xcd * each + (xcd < more ? xcd : more) + (blockIdx.x >> 3);
    const uint32_t tiles = (uint32_t)((a.nq + KT - 1) / KT);
    return make_int2((int)(w % tiles), (int)(w / tiles));
}

struct KnnLds {
    uint4 a[KT * KROW / 16], b[KT * KROW / 16];
    uint64_t buf[KT][KCAP];
    uint32_t cnt[KT];   // entries appended to buf (may exceed KCAP: the rest is offered again)
    uint32_t fill[KT];  // entries of the query's list
    uint32_t lim[KT];   // threshold: int / float bits, exclusive
    uint32_t t[KT];     // lim - |q|^2 (floats: knn_threshold)
    uint32_t qn[KT], bn[2 * KT];
    uint32_t again;
    uint32_t flag[3];   // of a step modulo 3: it has filled a buffer, nearly at least
};

// A chunk on its way to LDS: outside the rows or the vector the load has read another one (no branch holds it up), and
// zero takes its place; uint8 values are shifted by -128.
template <int DT>
__device__ __forceinline__ uint4 knn_stage(uint4 v, const bool in) {
    if (DT == JX_U8) {
        v.x ^= 0x80808080u;
        v.y ^= 0x80808080u;
        v.z ^= 0x80808080u;
        v.w ^= 0x80808080u;
    }
    return make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u);
}

// Four float32 values on their way to LDS as bfloat16: rounded, and what that leaves, rounded again.  Three parts: of the first
// sixteen coordinates
template <int PARTS>
__device__ __forceinline__ void knn_split(uint4* row, const int sch, const uint4 v) {
    float x[4] = {__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
    uint2 part[PARTS];
#pragma unroll
    for (int p = 0; p < PARTS; p++) {
        uint32_t h[2];
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const kf32x2 two = {x[2 * i], x[2 * i + 1]};
            h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, kbf16x2));
            x[2 * i] -= __uint_as_float(h[i] << 16);
            x[2 * i + 1] -= __uint_as_float(h[i] & 0xFFFF0000u);
        }
        part[p] = make_uint2(h[0], h[1]);
    }
#pragma unroll
    for (int p = 0; p < PARTS; p++) reinterpret_cast<uint2*>(row)[p * (PARTS == 3 ? 4 : 8) + sch] = part[p];
}

template <int DT>
__device__ __forceinline__ typename KAcc<DT>::elem knn_sq(uint4 v, typename KAcc<DT>::elem s) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if constexpr (DT == JX_U8)
            s = __builtin_amdgcn_sdot4((int)w[i], (int)w[i], s, false);
        else if constexpr (DT == JX_F16)
            s = hdot2(w[i], w[i], s);
        else
            s = fmaf(__uint_as_float(w[i]), __uint_as_float(w[i]), s);
    }
    return s;
}

template <int DT>
__device__ __forceinline__ uint32_t knn_bits(typename KAcc<DT>::elem v) {
    if constexpr (DT == JX_U8)
        return (uint32_t)v;
    else
        return __float_as_uint(v);
}
template <int DT>
__device__ __forceinline__ typename KAcc<DT>::elem knn_val(uint32_t b) {
    if constexpr (DT == JX_U8)
        return (int)b;
    else
        return __uint_as_float(b);
}

// A bound on the kp-th distance from what the slices have published for a query, plus one; 0x7F800000 if that is too little.
// Value r of a slice says that (r + 1) 2^pub_shift of its vectors are no farther, at any time (values only fall, in whatever
// order they are seen), so 2^pub_shift times the values <= t is at most the number of vectors within t: the need-th smallest
// value, need = ceil(kp / 2^pub_shift).  It is found by halving the range, 16 times at most: what is left above it, 2^-16 of
// the range, lets next to nothing in.  The largest r_th-th distance of the slices, which needs one value per slice, let in
// two to seven times as much: search launch of 1,000 x 100,003 float32 d = 960, k = 100 1,220 -> 1,136 us, of 10,000 x 1M
// uint8, k = 10 4,374 -> 3,998
struct KnnPublished {
    uint32_t v[KNN_ENTRIES / 64];
    // before other work: what takes its time is the way to memory that all XCDs see
    __device__ __forceinline__ void load(const uint32_t* published, const int entries, const int lane) {
#pragma unroll
        for (int r = 0; r < KNN_ENTRIES / 64; r++) {
            v[r] = 0x7F800000u;
            if (r * 64 < entries && r * 64 + lane < entries) v[r] = __hip_atomic_load(published + r * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
};
__device__ __forceinline__ uint32_t knn_limit(const KnnPublished& p, const int entries, const int need) {
    uint32_t lo = 0x7F800000u, hi = 0;
    int have = 0;
#pragma unroll
    for (int r = 0; r < KNN_ENTRIES / 64; r++) {
        if (r * 64 < entries) {  // uniform
            const bool on = p.v[r] < 0x7F800000u;
            have += __builtin_popcountll(ballot(on));
            lo = p.v[r] < lo ? p.v[r] : lo;
            hi = on && p.v[r] > hi ? p.v[r] : hi;
        }
    }
    if (have < need) return 0x7F800000u;
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
        const uint32_t l = shfl_xor(lo, x), h = shfl_xor(hi, x);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    lo = readlane32(lo, 0);
    hi = readlane32(hi, 0);
    for (int step = 0; step < 16 && lo < hi; step++) {
        const uint32_t mid = lo + (hi - lo) / 2;
        int c = 0;
#pragma unroll
        for (int r = 0; r < KNN_ENTRIES / 64; r++)
            if (r * 64 < entries) c += __builtin_popcountll(ballot(p.v[r] <= mid));
        if (c >= need) hi = mid;
        else lo = mid + 1;
    }
    return hi + 1u;  // equal distances stay in (their ids may be smaller)
}

// One wavefront merges the buffer of query row q into its list (sorted keys, kp at most) and renews the threshold.
// NL: list entries per lane.
template <int DT, int NL>
__device__ __forceinline__ void knn_flush(KnnLds& S, const int q, uint64_t* list, const int kp, uint32_t* published, const int nsplit,
                                          const int split, const int pub, const int shift, const int lane) {
    const int n_old = (int)S.fill[q];
    const int m = (int)S.cnt[q] < KCAP ? (int)S.cnt[q] : KCAP;
    KnnPublished others;
    if (published) others.load(published, nsplit * pub, lane);
    uint64_t old[NL];
    uint32_t to[NL];
#pragma unroll
    for (int r = 0; r < NL; r++) {
        const int p = r * 64 + lane;
        old[r] = p < n_old ? list[p] : JX_EMPTY_KEY;
        to[r] = (uint32_t)p;
    }
    const uint64_t mine = lane < m ? S.buf[q][lane] : JX_EMPTY_KEY;
    uint32_t at = 0;
    for (int i = 0; i < m; i++) {
        const uint64_t s = readlane64(mine, i);
        uint32_t rank = 0;
#pragma unroll
        for (int r = 0; r < NL; r++) {
            rank += (uint32_t)__builtin_popcountll(ballot(old[r] < s));
            to[r] += s < old[r] ? 1u : 0u;
        }
        at += (lane == i ? rank : 0u) + (s < mine ? 1u : 0u);
    }
    const int n_new = n_old + m < kp ? n_old + m : kp;
    uint32_t last = 0;  // distance of entry kp - 1
    bool has = false;
    auto place = [&](const uint64_t key, const uint32_t p) {
        const uint32_t dist = (uint32_t)(key >> 32);
        list[p] = key;
        if (p == (uint32_t)kp - 1u) {
            last = dist;
            has = true;
        }
        if (published && p < (uint32_t)(pub << shift) && ((p + 1) & ((1u << shift) - 1u)) == 0u)
            __hip_atomic_store(published + split * pub + (p >> shift), dist, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
#pragma unroll
    for (int r = 0; r < NL; r++)
        if (r * 64 + lane < n_old && to[r] < (uint32_t)kp) place(old[r], to[r]);
    if (lane < m && at < (uint32_t)kp) place(mine, at);
    __threadfence_block();  // the next merge of this list reads it with other lanes
    const uint64_t who = ballot(has);
    uint32_t lim = S.lim[q];
    if (who) {
        const uint32_t own = readlane32(last, __builtin_ctzll(who));
        if (own < lim) lim = own;  // ids of later steps are larger: a distance equal to the last one's is out
    }
    if (published) {
        const uint32_t all = knn_limit(others, nsplit * pub, (kp + (1 << shift) - 1) >> shift);
        if (all < lim) lim = all;
    }
    if (lane == 0) {
        S.lim[q] = lim;
        if constexpr (DT == JX_U8)
            S.t[q] = (uint32_t)((int)lim - (int)S.qn[q]);
        else
            S.t[q] = __float_as_uint(knn_threshold(__uint_as_float(lim), __uint_as_float(S.qn[q])));
        S.fill[q] = (uint32_t)n_new;
        S.cnt[q] = 0;
    }
    wave_sync();
}

// The first limits, a wavefront per query
__global__ void __launch_bounds__(64) knn_limit_kernel(KnnArgs a) {
    const long long qi = blockIdx.x;
    const int lane = threadIdx.x;
    KnnPublished p;
    p.load(a.published + (size_t)qi * a.nsplit * a.pub, a.nsplit * a.pub, lane);
    const uint32_t lim = knn_limit(p, a.nsplit * a.pub, (a.kp + (1 << a.pub_shift) - 1) >> a.pub_shift);
    if (lane == 0) a.redo[qi] = lim;
}

// Largest value of the wavefront, in every lane
template <typename E>
__device__ __forceinline__ E knn_wave_max(E v) {
    auto bits = [](E x) { return __builtin_bit_cast(uint32_t, x); };
    auto val = [](uint32_t x) { return __builtin_bit_cast(E, x); };
    auto top = [](E x, E y) { return x > y ? x : y; };
    v = top(v, val(dpp_u32<0xB1>(bits(v))));
    v = top(v, val(dpp_u32<0x4E>(bits(v))));
    v = top(v, val(dpp_u32<0x141>(bits(v))));
    v = top(v, val(dpp_u32<0x140>(bits(v))));
    return top(top(val(readlane32(bits(v), 0)), val(readlane32(bits(v), 16))), top(val(readlane32(bits(v), 32)), val(readlane32(bits(v), 48))));
}

// Whether the tiled kernel takes its tiles of 64 queries, first (.x) and second (.y) of this tile, whatever is found here:
// one query is hopeless on the word of all slices.  By a whole wavefront
__device__ __forceinline__ uint2 knn_hopeless(const KnnArgs& a, const long long tile, const int lane) {
    uint32_t w[4] = {~0u, ~0u, ~0u, ~0u};
    for (int s = lane; s < a.nsplit; s += 64) {
        const uint4 v = a.hopeless[tile * a.nsplit + s];
        w[0] &= v.x;
        w[1] &= v.y;
        w[2] &= v.z;
        w[3] &= v.w;
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        w[i] &= dpp_u32<0xB1>(w[i]);
        w[i] &= dpp_u32<0x4E>(w[i]);
        w[i] &= dpp_u32<0x141>(w[i]);
        w[i] &= dpp_u32<0x140>(w[i]);
        w[i] = readlane32(w[i], 0) & readlane32(w[i], 16) & readlane32(w[i], 32) & readlane32(w[i], 48);
    }
    return make_uint2(w[0] | w[1], w[2] | w[3]);
}

// What a seed launch publishes: best = largest 2 <q, b> - |b|^2 of each of the thread's 64 elements, 128 columns of a query in
// all; of the columns the first pub 2^pub_shift
template <int DT>
__device__ __forceinline__ void knn_publish(KnnLds& S, const KnnArgs& a, const typename KAcc<DT>::elem (&best)[64], const long long q0, const int split) {
    typedef typename KAcc<DT>::elem elem_t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, col = lane & 31, half = lane >> 5;
    elem_t* cols = reinterpret_cast<elem_t*>(&S.buf[0][0]);  // [64][128]
    static_assert(sizeof(S.buf) >= 64 * 128 * 4, "columns of 64 queries");
    for (int h = 0; h < 2; h++) {  // 64 queries at a time
        if (wm == h) {
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++)
#pragma unroll
                    for (int e = 0; e < 16; e++)
                        cols[(i * 32 + 8 * (e >> 2) + 4 * half + (e & 3)) * 128 + wn * 64 + j * 32 + col] = best[(i * 2 + j) * 16 + e];
        }
        __syncthreads();
        for (int r = wave; r < 64; r += 4) {
            const long long qi = q0 + h * 64 + r;
            if (qi >= a.nq) break;
            elem_t x = cols[r * 128 + lane], y = cols[r * 128 + 64 + lane];
            const elem_t none = DT == JX_U8 ? (elem_t)-0x7FFFFFFF : (elem_t)-__builtin_inff();
            const elem_t qn = knn_val<DT>(S.qn[h * 64 + r]);
            for (int k = 0; k < a.pub << a.pub_shift; k++) {
                const elem_t m = knn_wave_max<elem_t>(x > y ? x : y);
                const uint64_t hx = ballot(x == m), hy = ballot(y == m);
                if (hx) {
                    if (lane == __builtin_ctzll(hx)) x = none;
                } else if (hy) {
                    if (lane == __builtin_ctzll(hy)) y = none;
                }
                uint32_t code = 0x7F800000u;
                if constexpr (DT == JX_U8) {
                    if (m > -0x40000000) code = (uint32_t)(qn - m);
                } else {
                    const float d = fmaxf(qn - m, 0.f);
                    if (d < __builtin_inff() && m > -__builtin_inff()) code = __float_as_uint(d);
                }
                if (lane == 0) {
                    if (((k + 1) & ((1 << a.pub_shift) - 1)) == 0) a.published[((size_t)qi * a.nsplit + split) * a.pub + (k >> a.pub_shift)] = code;
                    if (k == a.r_th - 1) S.lim[h * 64 + r] = code;
                }
            }
        }
        __syncthreads();
    }
}

// SEED: only the slice's first a.seed_steps steps, to publish a first r_th distance before the search begins: the
// smallest distance of each of the 128 columns over the steps, then the r_th smallest of these.  It is no smaller than
// the r_th of all that was seen.  Float types: a query whose distances can be off by more than a share of that first
// distance (a set far from the origin, squares that are subnormal) will hardly be proven: the KNN_SLACK candidates behind the
// k-th would have to reach as far beyond it.  Where each half of a tile holds such a query the tiled kernel runs for all of
// it anyway, and this one stops here.  The share is a quarter of the slack's part of the list, 0.24 at k = 1, 0.18 at 10 and
// 0.05 at 100; a set of 16 intrinsic dimensions has 0.34, 0.15 and 0.03 between the k-th and the last.
// 1,000 from the origin, k = 10, with the stop / without / the tiled kernel alone: 256 x 100,003 float32 d = 960 4,330 / 5,190
// / 4,216 us, 1,000 x 200,000 float32 d = 128 1,893 / 3,270 / 1,822, 256 x 100,000 binary16 d = 960 1,891 / 2,298 / 1,817.
// What only the finished lists show is paid twice: 29 or more copies of every vector 5,103 / 4,216 and 2,971 / 1,860
//
// FEW: float32 of at most KNN_FEW_D dimensions, one slab of sixteen coordinates in three parts: the six matrix instructions that
// two parts of 32 coordinates take, half the rows to stage and the queries' staged once.  With two parts vectors of few dimensions
// that lie far from the origin cannot be proven.  k = 10, two parts / three / float32 instruction (which could prove them): d = 4
// ten standard deviations away 1,000 x 100,000 722 / 200 / 561 us, 1,000 x 1M 2,240 / 685 / 1,876, 32 x 200,000 612 / 90 / 318;
// d = 16 around the origin 217 / 205 / 569, 800 / 690 / 1,880 and 97 / 89 / 320
template <int DT, int NL, bool SEED, bool FEW = false>
__global__ void __launch_bounds__(256, 2) knn_tile_kernel(KnnArgs a) {
    constexpr int PARTS = FEW ? 3 : 2;
    constexpr int TPR = FEW ? 4 : 8, NT = KT * TPR / 256, STEP = 256 / TPR;  // staging: threads per row, rows per thread and how far apart
    typedef typename KAcc<DT>::type acc_t;
    typedef typename KAcc<DT>::elem elem_t;
    __shared__ KnnLds S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, col = lane & 31, half = lane >> 5;
    const int2 work = knn_work(a);
    const int tile = work.x, split = work.y;
    const long long q0 = (long long)tile * KT;
    const long long steps = (a.n + KT - 1) / KT;  // every slice has as many, or one more
    const long long b_begin = split * steps / a.nsplit * KT;
    long long b_end = (split + 1) * steps / a.nsplit * KT;
    if (b_end > a.n) b_end = a.n;
    if (SEED && b_end > b_begin + (long long)a.seed_steps * KT) b_end = b_begin + (long long)a.seed_steps * KT;
    const uint8_t* Q = reinterpret_cast<const uint8_t*>(a.queries);
    const uint8_t* B = reinterpret_cast<const uint8_t*>(a.base);
    const int nslab = (a.nch + 7) / 8;
    const int srow = tid / TPR, sch = tid % TPR;

    for (int i = tid; i < KT; i += 256) {
        S.cnt[i] = 0;
        S.fill[i] = 0;
        uint32_t lim = DT == JX_U8 ? (uint32_t)KINF : 0x7F800000u;
        if (!SEED && a.seed_steps && q0 + i < a.nq) {
            const uint32_t first = a.redo[q0 + i];
            if (first < lim) lim = first;
        }
        S.lim[i] = lim;
    }
    if constexpr (DT != JX_U8 && !SEED) {
        if (a.seed_steps) {
            const uint2 w = knn_hopeless(a, tile, lane);
            if (w.x && (w.y || q0 + 64 >= a.nq)) return;  // the whole workgroup
        }
    }
    if (tid == 0) S.again = 0;
    if (SEED && DT != JX_U8 && split == 0 && tid < 2) (&a.odd[tile].count)[tid] = 0u;  // count and bb_max
    __syncthreads();
    elem_t best[SEED ? 64 : 1];  // largest 2 <q, b> - |b|^2 of each element
    if constexpr (SEED) {
#pragma unroll
        for (int e = 0; e < 64; e++) best[e] = DT == JX_U8 ? (elem_t)-0x7FFFFFFF : (elem_t)-__builtin_inff();
    }
    uint32_t bmax = 0;

    uint4 pa[NT], pb[NT];
    const size_t row_bytes = (size_t)(a.nch * 16);
    auto at = [&](const uint8_t* base, const long long row, const long long rows, const int ch) {
        return load16(base + (size_t)(row < rows ? row : rows - 1) * row_bytes + (size_t)((ch < a.nch ? ch : a.nch - 1) * 16));
    };
    auto fetch = [&](const long long b0, const int slab) {
#pragma unroll
        for (int t = 0; t < NT; t++) pb[t] = at(B, b0 + srow + STEP * t, b_end, slab * 8 + sch);
#pragma unroll
        for (int t = 0; t < NT; t++)
            if (!FEW || b0 == b_begin) pa[t] = at(Q, q0 + srow + STEP * t, a.nq, slab * 8 + sch);
    };
    if (b_begin < b_end) fetch(b_begin, 0);

    for (long long b0 = b_begin; b0 < b_end; b0 += KT) {
        const bool first = b0 == b_begin;
        acc_t acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[i][j][e] = 0;
        elem_t nb[NT] = {}, nq[NT] = {};
        for (int slab = 0; slab < nslab; slab++) {
#pragma unroll
            for (int t = 0; t < NT; t++) {
                const bool chunk = slab * 8 + sch < a.nch;
                if (!FEW || first) {
                    const uint4 v = knn_stage<DT>(pa[t], chunk && q0 + srow + STEP * t < a.nq);
                    if constexpr (DT == JX_F32)
                        knn_split<PARTS>(S.a + (srow + STEP * t) * (KROW / 16), sch, v);
                    else
                        S.a[(srow + STEP * t) * (KROW / 16) + sch] = v;
                    if (first) nq[t] = knn_sq<DT>(v, nq[t]);
                }
                const uint4 v = knn_stage<DT>(pb[t], chunk && b0 + srow + STEP * t < b_end);
                if constexpr (DT == JX_F32)
                    knn_split<PARTS>(S.b + (srow + STEP * t) * (KROW / 16), sch, v);
                else
                    S.b[(srow + STEP * t) * (KROW / 16) + sch] = v;
                nb[t] = knn_sq<DT>(v, nb[t]);
            }
            if (slab == nslab - 1) {  // norms: the threads of a row
                uint32_t norm[NT];
#pragma unroll
                for (int t = 0; t < NT; t++) {
                    const int row = srow + STEP * t;
                    const elem_t x = group_sum<TPR>(nb[t]);
                    const bool in = b0 + row < b_end;
                    norm[t] = in ? knn_bits<DT>(x) : 0u;
                    // binary16: what is listed as odd takes no other way into the result
                    if (sch == 0) S.bn[row] = DT == JX_F16 && norm[t] == 0x7F800000u ? 0x7FC00000u : (in ? norm[t] : (DT == JX_U8 ? 0x7FFFFFFFu : 0x7F800000u));
                    if (first) {
                        const elem_t y = group_sum<TPR>(nq[t]);
                        if (sch == 0) {
                            S.qn[row] = knn_bits<DT>(y);
                            // rows beyond the last query accept nothing
                            if (DT == JX_U8)
                                S.t[row] = q0 + row < a.nq ? (uint32_t)((int)S.lim[row] - (int)y) : 0xB0000000u;
                            else if (S.lim[row] < 0x7F800000u)
                                S.t[row] = q0 + row < a.nq ? __float_as_uint(knn_threshold(__uint_as_float(S.lim[row]), (float)y)) : 0xFF800000u;
                            else
                                S.t[row] = q0 + row < a.nq ? 0x7F800000u : 0xFF800000u;
                        }
                    }
                }
                if constexpr (DT != JX_U8 && !SEED) {
                    const uint32_t most = NT == 2 ? max(norm[0], norm[1]) : max(max(norm[0], norm[1]), max(norm[NT - 2], norm[NT - 1]));
                    if (most < KNN_DECIDABLE<DT>) {
                        bmax = max(bmax, most);
                    } else if (sch == 0) {
#pragma unroll
                        for (int t = 0; t < NT; t++) {
                            if (norm[t] < KNN_DECIDABLE<DT>) {
                                bmax = max(bmax, norm[t]);
                            } else {
                                const uint32_t to = atomicAdd(&a.odd[tile].count, 1u);
                                if (to < KNN_ODD) a.odd[tile].id[to] = (uint32_t)(b0 + srow + STEP * t);
                            }
                        }
                    }
                }
            }
            __syncthreads();
            if (slab + 1 < nslab)
                fetch(b0, slab + 1);
            else if (b0 + KT < b_end)
                fetch(b0 + KT, 0);
            if constexpr (FEW) {
                kbf16x8 fb[2][3];  // [tile][part]
#pragma unroll
                for (int j = 0; j < 2; j++)
#pragma unroll
                    for (int p = 0; p < 3; p++) fb[j][p] = __builtin_bit_cast(kbf16x8, S.b[(wn * 64 + j * 32 + col) * (KROW / 16) + p * 2 + half]);
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    kbf16x8 fa[3];
#pragma unroll
                    for (int p = 0; p < 3; p++) fa[p] = __builtin_bit_cast(kbf16x8, S.a[(wm * 64 + i * 32 + col) * (KROW / 16) + p * 2 + half]);
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[2], fb[j][0], acc[i][j], 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[j][2], acc[i][j], 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[j][1], acc[i][j], 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[j][0], acc[i][j], 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[j][1], acc[i][j], 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[j][0], acc[i][j], 0, 0, 0);
                    }
                }
            } else if constexpr (DT == JX_F32) {
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    kbf16x8 fa[2][2], fb[2][2];  // [tile][part]
#pragma unroll
                    for (int i = 0; i < 2; i++)
#pragma unroll
                        for (int p = 0; p < 2; p++) {
                            fa[i][p] = __builtin_bit_cast(kbf16x8, S.a[(wm * 64 + i * 32 + col) * (KROW / 16) + p * 4 + s * 2 + half]);
                            fb[i][p] = __builtin_bit_cast(kbf16x8, S.b[(wn * 64 + i * 32 + col) * (KROW / 16) + p * 4 + s * 2 + half]);
                        }
#pragma unroll
                    for (int i = 0; i < 2; i++)
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][1], fb[j][0], acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][0], fb[j][1], acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][0], fb[j][0], acc[i][j], 0, 0, 0);
                        }
                }
            } else {
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    uint4 fa[2], fb[2];
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        fa[i] = S.a[(wm * 64 + i * 32 + col) * (KROW / 16) + s * 2 + half];
                        fb[i] = S.b[(wn * 64 + i * 32 + col) * (KROW / 16) + s * 2 + half];
                    }
#pragma unroll
                    for (int i = 0; i < 2; i++)
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            if constexpr (DT == JX_U8)
                                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(ki32x4, fa[i]), __builtin_bit_cast(ki32x4, fb[j]), acc[i][j], 0, 0, 0);
                            else
                                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(kf16x8, fa[i]), __builtin_bit_cast(kf16x8, fb[j]), acc[i][j], 0, 0, 0);
                        }
                }
            }
            if (slab + 1 < nslab) __syncthreads();  // else the barrier behind the appends stands before the next write
        }
        elem_t nbv[2];
#pragma unroll
        for (int j = 0; j < 2; j++) nbv[j] = knn_val<DT>(S.bn[wn * 64 + j * 32 + col]);
        if constexpr (SEED) {
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++)
#pragma unroll
                    for (int e = 0; e < 16; e++) {
                        const elem_t v = acc[i][j][e] * 2 - nbv[j];
                        elem_t& m = best[(i * 2 + j) * 16 + e];
                        m = v > m ? v : m;
                    }
            __syncthreads();
            continue;
        }
        // ---- compare and append; what found a full buffer is offered again after the merges
        uint64_t stored = 0;  // elements of this lane's 64 that are in a buffer already
        for (int round = 0;; round++) {
#pragma unroll
            for (int i = 0; i < 2; i++) {
                uint4 tv[4];
#pragma unroll
                for (int h = 0; h < 4; h++) tv[h] = *reinterpret_cast<const uint4*>(&S.t[wm * 64 + i * 32 + 8 * h + 4 * half]);
#pragma unroll
                for (int h = 0; h < 4; h++) {
                    int r0 = wm * 64 + i * 32 + 8 * h + 4 * half;
                    asm volatile("" : "+v"(r0));  // not known outside: addresses of all 64 elements would not fit the registers
                    const uint32_t tt[4] = {tv[h].x, tv[h].y, tv[h].z, tv[h].w};
                    // d < limit as 2 <q, b> + t > |b|^2, t = limit - |q|^2: the largest of four rows first
                    elem_t v[2][4];
                    bool any = false;
#pragma unroll
                    for (int j = 0; j < 2; j++) {
#pragma unroll
                        for (int c = 0; c < 4; c++) {
                            const elem_t x = acc[i][j][h * 4 + c], t = knn_val<DT>(tt[c]);
                            if constexpr (DT == JX_U8)
                                v[j][c] = (x << 1) + t;
                            else
                                v[j][c] = fmaf(2.f, x, t);
                        }
                        elem_t most;
                        if constexpr (DT == JX_U8)
                            most = max(max(max(v[j][0], v[j][1]), v[j][2]), v[j][3]);
                        else
                            most = fmaxf(fmaxf(fmaxf(v[j][0], v[j][1]), v[j][2]), v[j][3]);
                        any = any || most >= nbv[j];
                    }
                    if (ballot(any) == 0ull) continue;
#pragma unroll
                    for (int c = 0; c < 4; c++)
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            const int bit = ((i * 4 + h) * 4 + c) * 2 + j;
                            const uint32_t id = (uint32_t)b0 + (uint32_t)(wn * 64 + j * 32 + col);
                            if ((round == 0 ? v[j][c] > nbv[j] : v[j][c] >= nbv[j]) && !((stored >> bit) & 1ull) && id < (uint32_t)b_end) {
                                const uint32_t pos = atomicAdd(&S.cnt[r0 + c], 1u);
                                if (pos < KCAP) {
                                    uint32_t code;
                                    const elem_t x = acc[i][j][h * 4 + c], qn = knn_val<DT>(S.qn[r0 + c]);
                                    if constexpr (DT == JX_U8)
                                        code = (uint32_t)(qn + nbv[j] - 2 * x);
                                    else
                                        code = __float_as_uint(fmaxf((qn + nbv[j]) - 2.f * x, 0.f));
                                    S.buf[r0 + c][pos] = ((uint64_t)code << 32) | (uint64_t)id;
                                    stored |= 1ull << bit;
                                } else {
                                    S.again = 1;
                                }
                            }
                        }
                }
            }
            __syncthreads();
            const uint32_t again = S.again;
            // wavefront w merges the buffers of rows 32 w .. 32 w + 31
            uint64_t need = ballot(lane < 32 && S.cnt[wave * 32 + (lane & 31)] >= KFLUSH);
            while (need) {
                const int q = wave * 32 + __builtin_ctzll(need);
                need &= need - 1ull;
                knn_flush<DT, NL>(S, q, a.lists + ((size_t)(q0 + q) * a.nsplit + split) * a.kp, a.kp,
                                   a.published ? a.published + (size_t)(q0 + q) * a.nsplit * a.pub : nullptr, a.nsplit, split, a.pub,
                                   a.pub_shift, lane);
            }
            if (!again) break;  // the next step's first barrier stands between these merges and its appends
            __syncthreads();
            if (tid == 0) S.again = 0;
            __syncthreads();
        }
    }
    if constexpr (SEED) {
        knn_publish<DT>(S, a, best, q0, split);
        if constexpr (DT != JX_U8) {
            if (tid < KT) {
                const float first = __uint_as_float(S.lim[tid]);
                const bool hope = first < __builtin_inff() && knn_eps(a.d, __uint_as_float(S.qn[tid]), first, __builtin_inff(), a.parts) * (float)a.kp <= first * (float)(KNN_SLACK / 4);
                const uint64_t bits = ballot(q0 + tid < a.nq && !hope);
                if (lane == 0) reinterpret_cast<uint64_t*>(a.hopeless + (size_t)tile * a.nsplit + split)[wave] = bits;
            }
        }
        return;
    }
    // ---- what is left in the buffers, and the padding of short lists
    __syncthreads();
    for (int i = 0; i < 32; i++) {
        const int q = wave * 32 + i;
        if (q0 + q >= a.nq) break;
        uint64_t* list = a.lists + ((size_t)(q0 + q) * a.nsplit + split) * a.kp;
        if (S.cnt[q]) knn_flush<DT, NL>(S, q, list, a.kp, nullptr, 0, 0, 0, 0, lane);
        for (int e = (int)S.fill[q] + lane; e < a.kp; e += 64) list[e] = JX_EMPTY_KEY;
    }
    if (DT != JX_U8) {
        __syncthreads();
        if (tid == 0) S.again = 0;
        __syncthreads();
        atomicMax(&S.again, bmax);
        __syncthreads();
        if (tid == 0) atomicMax(&a.odd[tile].bb_max, S.again);
    }
}

// uint8 vectors of at most 128 bytes: one slab.  What a step costs besides its 16 matrix instructions a wavefront is
// vector instructions and barriers, so:
//   the queries' operands stay in registers;
//   an accumulator starts at (t + 1) / 2, t = limit - |q|^2 of its query, as the first matrix instruction's C operand, so
//   that the test 2 <q, b> + t > |b|^2 is one comparison of the largest of 16 elements with |b|^2 / 2 (rounded down: what
//   passes is looked at again, exactly);
//   the base vectors are staged in two buffers, and the only barrier of a step stands between staging and use.  What the
//   step before has appended is merged behind that barrier, its accumulators still at hand for what found a full buffer.
// 342 -> 235 vector instructions a step, appends and merges included; search launch of 10,000 x 1M, d = 128, k = 10
// 3,998 -> 3,233 us, without a single candidate 3,056 -> 2,000 (the int8 rate of a large product: 1,239).
template <int NL, bool SEED>
__global__ void __launch_bounds__(256, 2) knn_u8_kernel(KnnArgs a) {
    __shared__ KnnLds S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, col = lane & 31, half = lane >> 5;
    const uint32_t tiles = (uint32_t)((a.nq + KT - 1) / KT);
    const long long q0 = (long long)(blockIdx.x % tiles) * KT;
    const int split = (int)(blockIdx.x / tiles);
    knn_row b_begin, b_end;
    knn_slice(a.n, a.nsplit, split, &b_begin, &b_end);
    b_begin = (knn_row)__builtin_amdgcn_readfirstlane((int)b_begin);
    b_end = (knn_row)__builtin_amdgcn_readfirstlane((int)b_end);
    if (SEED && b_end - b_begin > (knn_row)a.seed_steps * KT) b_end = b_begin + (knn_row)a.seed_steps * KT;
    const uint8_t* Q = reinterpret_cast<const uint8_t*>(a.queries);
    const uint8_t* B = reinterpret_cast<const uint8_t*>(a.base);
    const int srow = tid >> 3, sch = tid & 7;  // staging: 8 threads per row, rows srow + 32 t
    const size_t row_bytes = (size_t)(a.nch * 16);
    const bool whole = a.nch == 8;

    for (int i = tid; i < KT; i += 256) {
        S.cnt[i] = 0;
        S.fill[i] = 0;
        uint32_t lim = (uint32_t)KINF;
        if (!SEED && a.seed_steps && q0 + i < a.nq) {
            const uint32_t first = a.redo[q0 + i];
            if (first < lim) lim = first;
        }
        S.lim[i] = lim;
    }
    if (tid < 3) S.flag[tid] = 0;
    if (tid == 0) S.again = 0;
    __syncthreads();
    ki32x4 fa[2][4];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int row = wm * 64 + i * 32 + col;
        const bool in = q0 + row < a.nq;
        int nn = 0;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const int ch = s * 2 + half;
            const uint4 v = knn_stage<JX_U8>(load16(Q + (size_t)(in ? q0 + row : q0) * row_bytes + (size_t)((ch < a.nch ? ch : 0) * 16)), in && ch < a.nch);
            nn = knn_sq<JX_U8>(v, nn);
            fa[i][s] = __builtin_bit_cast(ki32x4, v);
        }
        nn += shfl_xor(nn, 32);
        if (wn == 0 && half == 0) {
            S.qn[row] = (uint32_t)nn;
            S.t[row] = in ? (uint32_t)((int)S.lim[row] - nn) : 0xB0000000u;  // rows beyond the last query accept nothing
        }
    }
    __syncthreads();
    ki32x16 start[2];  // the accumulators' first values
    auto load_start = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int h = 0; h < 4; h++) {
                const int4 t = *reinterpret_cast<const int4*>(&S.t[wm * 64 + i * 32 + 8 * h + 4 * half]);
                start[i][4 * h] = (t.x + 1) >> 1;
                start[i][4 * h + 1] = (t.y + 1) >> 1;
                start[i][4 * h + 2] = (t.z + 1) >> 1;
                start[i][4 * h + 3] = (t.w + 1) >> 1;
            }
    };
    if (!SEED) load_start();
    int best[SEED ? 64 : 1];
#pragma unroll
    for (int e = 0; e < (SEED ? 64 : 1); e++) best[e] = -0x7FFFFFFF;
    uint4 pb[4];
    auto fetch = [&](const knn_row b0) __attribute__((always_inline)) {
        if (knn_whole_step(b0, b_end) && whole) {  // uniform
#pragma unroll
            for (int t = 0; t < 4; t++) pb[t] = load16(B + (size_t)(b0 + srow + 32 * t) * 128 + sch * 16);
        } else {
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const knn_row row = b0 + srow + 32 * t;
                pb[t] = load16(B + (size_t)(row < b_end ? row : b_end - 1) * row_bytes + (size_t)((sch < a.nch ? sch : 0) * 16));
            }
        }
    };
    if (b_begin < b_end) fetch(b_begin);
    ki32x16 acc[2][2];
    uint64_t stored = 0;
    // Appends what of a step passes; a full buffer leaves the element for the next round (later rounds: limits may have come
    // down to a distance that an element stored in the meantime has, and equal ones stay in)
    auto append = [&](const knn_row b0, const int cur, const int slot, const bool again) __attribute__((always_inline)) {
        int nbv[2];
#pragma unroll
        for (int j = 0; j < 2; j++) nbv[j] = (int)S.bn[cur * KT + wn * 64 + j * 32 + col];
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int h = 0; h < 4; h++) {
                int r0 = wm * 64 + i * 32 + 8 * h + 4 * half;
                asm volatile("" : "+v"(r0));  // not known outside: addresses of all 64 elements would not fit the registers
                int most[2];
#pragma unroll
                for (int j = 0; j < 2; j++) most[j] = max(max(max(acc[i][j][4 * h], acc[i][j][4 * h + 1]), acc[i][j][4 * h + 2]), acc[i][j][4 * h + 3]);
                if (!again && ballot(most[0] > (nbv[0] >> 1) || most[1] > (nbv[1] >> 1)) == 0ull) continue;
                const int4 t4 = *reinterpret_cast<const int4*>(&S.t[r0]);
                const int tt[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                for (int c = 0; c < 4; c++)
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        const int bit = ((i * 4 + h) * 4 + c) * 2 + j;
                        const knn_row id = b0 + (knn_row)(wn * 64 + j * 32 + col);
                        const int x = acc[i][j][h * 4 + c] - start[i][h * 4 + c];
                        const int v = (x << 1) + tt[c];
                        if ((again ? v >= nbv[j] : v > nbv[j]) && !((stored >> bit) & 1ull) && id < b_end) {
                            const uint32_t pos = atomicAdd(&S.cnt[r0 + c], 1u);
                            if (pos < KCAP) {
                                S.buf[r0 + c][pos] = ((uint64_t)(uint32_t)((int)S.qn[r0 + c] + nbv[j] - 2 * x) << 32) | (uint64_t)id;
                                stored |= 1ull << bit;
                            } else {
                                S.again = 1;
                            }
                            if (pos >= KFLUSH - 1) S.flag[slot] = 1;
                        }
                    }
            }
    };
    int cur = 0, slot = 0;  // staging buffer and flag of the step
    for (knn_row b0 = b_begin;; b0 += KT, cur ^= 1, slot = slot == 2 ? 0 : slot + 1) {
        uint4* stage = cur ? S.b : S.a;
        if (b0 < b_end) {
            const bool full = knn_whole_step(b0, b_end) && whole;  // uniform
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const int row = srow + 32 * t;
                const bool in = b0 + row < b_end;
                const uint4 v = full ? knn_stage<JX_U8>(pb[t], true) : knn_stage<JX_U8>(pb[t], in && sch < a.nch);
                stage[row * (KROW / 16) + sch] = v;
                const int nn = group_sum<8>(knn_sq<JX_U8>(v, 0));
                if (sch == 0) S.bn[cur * KT + row] = in ? (uint32_t)nn : 0x7FFFFFFFu;
            }
        }
        __syncthreads();
        const int before = slot == 0 ? 2 : slot - 1;
        if (!SEED && S.flag[before]) {  // the same in every thread: written before the barrier, cleared behind the next
            // the step before: merge its buffers that are nearly full, and offer again what found a full one
            for (;;) {
                // wavefront w merges the buffers of rows 32 w .. 32 w + 31
                uint64_t need = ballot(lane < 32 && S.cnt[wave * 32 + (lane & 31)] >= KFLUSH);
                while (need) {
                    const int q = wave * 32 + __builtin_ctzll(need);
                    need &= need - 1ull;
                    knn_flush<JX_U8, NL>(S, q, a.lists + ((size_t)(q0 + q) * a.nsplit + split) * a.kp, a.kp,
                                         a.published ? a.published + (size_t)(q0 + q) * a.nsplit * a.pub : nullptr, a.nsplit, split, a.pub,
                                         a.pub_shift, lane);
                }
                __syncthreads();
                const uint32_t more = S.again;
                __syncthreads();
                if (!more) break;
                if (tid == 0) S.again = 0;
                __syncthreads();
                append(b0 - KT, cur ^ 1, before, true);
                __syncthreads();
            }
            load_start();
        }
        if (b0 >= b_end) break;
        if (tid == 0) S.flag[slot == 2 ? 0 : slot + 1] = 0;  // the next step's: last read before the barrier above
        if (!knn_last_step(b0, b_end)) fetch(b0 + KT);
        if constexpr (SEED) {
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int e = 0; e < 16; e++) start[i][e] = 0;
        }
        const uint4* opnd = stage + (wn * 64 + col) * (KROW / 16) + half;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            ki32x4 fb[2];
#pragma unroll
            for (int j = 0; j < 2; j++) fb[j] = __builtin_bit_cast(ki32x4, opnd[j * 32 * (KROW / 16) + s * 2]);
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i][s], fb[j], s ? acc[i][j] : start[i], 0, 0, 0);
        }
        if constexpr (SEED) {
#pragma unroll
            for (int j = 0; j < 2; j++) {
                const int nb = (int)S.bn[cur * KT + wn * 64 + j * 32 + col];
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int e = 0; e < 16; e++) best[(i * 2 + j) * 16 + e] = max(best[(i * 2 + j) * 16 + e], (acc[i][j][e] << 1) - nb);
            }
            continue;
        }
        bool any = false;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int nbh = (int)S.bn[cur * KT + wn * 64 + j * 32 + col] >> 1;
#pragma unroll
            for (int i = 0; i < 2; i++) {
                int most = acc[i][j][0];
#pragma unroll
                for (int e = 1; e < 16; e++) most = max(most, acc[i][j][e]);
                any = any || most > nbh;
            }
        }
        stored = 0;
        if (ballot(any)) append(b0, cur, slot, false);
    }
    if constexpr (SEED) {
        knn_publish<JX_U8>(S, a, best, q0, split);
        return;
    }
    // ---- what is left in the buffers, and the padding of short lists
    for (int i = 0; i < 32; i++) {
        const int q = wave * 32 + i;
        if (q0 + q >= a.nq) break;
        uint64_t* list = a.lists + ((size_t)(q0 + q) * a.nsplit + split) * a.kp;
        if (S.cnt[q]) knn_flush<JX_U8, NL>(S, q, list, a.kp, nullptr, 0, 0, 0, 0, lane);
        for (int e = (int)S.fill[q] + lane; e < a.kp; e += 64) list[e] = JX_EMPTY_KEY;
    }
}

// One wavefront per query: the kp smallest keys of its lists, then (float types) the exact distances.
template <int DT, int NL>
__global__ void __launch_bounds__(64) knn_merge_kernel(KnnArgs a) {
    __shared__ uint64_t ex[(NL + 1) * 64];
    const long long qi = blockIdx.x;
    const int lane = threadIdx.x;
    const int kp = a.kp;
    int nlists = a.nsplit;
    if constexpr (DT != JX_U8) {
        if (a.seed_steps) {
            const uint2 w = knn_hopeless(a, qi / KT, lane);
            if (qi % KT < 64 ? w.x : w.y) nlists = 0;  // there may be none; the result stays unproven
        }
    }
    uint64_t top[NL];
#pragma unroll
    for (int r = 0; r < NL; r++) top[r] = JX_EMPTY_KEY;
    uint64_t worst = JX_EMPTY_KEY;  // entry kp - 1
    const uint64_t* src = a.lists + (size_t)qi * a.nsplit * kp;
    for (int s0 = 0; s0 < nlists; s0 += 64) {  // a list per lane, entry by entry
        for (int c = 0; c < kp; c++) {
            const uint64_t key = s0 + lane < nlists ? src[(size_t)(s0 + lane) * kp + c] : JX_EMPTY_KEY;
            uint64_t todo = ballot(key < worst);
            if (todo == 0ull) break;  // the lists are sorted: what follows is no smaller
            while (todo) {
                const uint64_t x = readlane64(key, __builtin_ctzll(todo));
                todo &= todo - 1ull;
                int rank = 0;
#pragma unroll
                for (int r = 0; r < NL; r++) rank += __builtin_popcountll(ballot(top[r] < x));
#pragma unroll
                for (int r = NL - 1; r >= 0; r--) {
                    const uint64_t in = r ? readlane64(top[r ? r - 1 : 0], 63) : 0ull;
                    const uint64_t up = wave_shift_up(top[r], in);
                    const int p = r * 64 + lane;
                    top[r] = p < rank ? top[r] : (p == rank ? x : up);
                }
            }
#pragma unroll
            for (int r = 0; r < NL; r++) {
                if (r * 64 + lane >= kp) top[r] = JX_EMPTY_KEY;
                if (r == (kp - 1) >> 6) worst = readlane64(top[r], (kp - 1) & 63);
            }
        }
    }
    if constexpr (DT == JX_U8) {
#pragma unroll
        for (int r = 0; r < NL; r++) {
            const int p = r * 64 + lane;
            if (p < a.k) {
                const bool valid = top[r] != JX_EMPTY_KEY;
                a.out_ids[qi * a.k + p] = valid ? (uint32_t)top[r] : JX_NONE_ID;
                a.out_dist[qi * a.k + p] = valid ? (float)(uint32_t)(top[r] >> 32) : __builtin_inff();
            }
        }
        return;
    }
    // ---- the distances of bruteforce_tile_kernel: one candidate per lane, the same operations in the same order.  Nothing is
    // stored to global memory on any path before: the query's loads would no longer be scalar ones (1,000 queries of d = 960,
    // 128 candidates 136 -> 187 us)
    const uint4* q4 = reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(a.queries) + (size_t)qi * (size_t)(a.nch * 16));
    float qq = 0.f;  // |q|^2: binary16 in that kernel's order, float32 only for the bound
    for (int ch = 0; ch < a.nch; ch++) qq = knn_sq<DT>(q4[ch], qq);
    const KnnOdd& odd = a.odd[qi / KT];
    const int n_odd = odd.count < KNN_ODD ? (int)odd.count : KNN_ODD;
    int n_valid = 0;
    // the list's candidates, then the rows that are in no list
    for (int r = 0; r <= NL; r++) {
        uint64_t cur = r == NL && lane < n_odd ? (uint64_t)odd.id[lane < KNN_ODD ? lane : 0] : JX_EMPTY_KEY;
#pragma unroll
        for (int x = 0; x < NL; x++)
            if (x == r) cur = top[x];
        const bool valid = cur != JX_EMPTY_KEY;
        const uint64_t vm = ballot(valid);
        if (vm == 0ull) continue;
        const uint32_t id = valid ? (uint32_t)cur : 0u;
        const uint4* b4 = reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(a.base) + (size_t)id * (size_t)(a.nch * 16));
        float acc = 0.f, bb = 0.f;
#pragma unroll 8
        for (int ch = 0; ch < a.nch; ch++) {
            const uint4 x = q4[ch], y = b4[ch];
            if constexpr (DT == JX_F16) {
                acc = hdot2(x.x, y.x, acc);
                acc = hdot2(x.y, y.y, acc);
                acc = hdot2(x.z, y.z, acc);
                acc = hdot2(x.w, y.w, acc);
                bb = knn_sq<DT>(y, bb);
            } else {
                float d;
                d = __uint_as_float(x.x) - __uint_as_float(y.x);
                acc = fmaf(d, d, acc);
                d = __uint_as_float(x.y) - __uint_as_float(y.y);
                acc = fmaf(d, d, acc);
                d = __uint_as_float(x.z) - __uint_as_float(y.z);
                acc = fmaf(d, d, acc);
                d = __uint_as_float(x.w) - __uint_as_float(y.w);
                acc = fmaf(d, d, acc);
            }
        }
        const float dist = DT == JX_F16 ? fmaxf(qq + bb - 2.f * acc, 0.f) : acc;
        if (valid) ex[n_valid + lane] = ((uint64_t)f32_to_ordered(dist) << 32) | id;
        n_valid += __builtin_popcountll(vm);
    }
    for (int p = n_valid + lane; p < (NL + 1) * 64; p += 64) ex[p] = JX_EMPTY_KEY;
    wave_sync();
    float kth = -1.f;
    for (int r = 0; r * 64 < n_valid; r++) {
        const uint64_t mine = ex[r * 64 + lane];
        int rank = 0;
        for (int t = 0; t < n_valid; t++) rank += ex[t] < mine ? 1 : 0;
        if (mine != JX_EMPTY_KEY && rank < a.k) {
            const float dist = ordered_to_f32((uint32_t)(mine >> 32));
            a.out_ids[qi * a.k + rank] = (uint32_t)mine;
            a.out_dist[qi * a.k + rank] = dist;
            if (rank == a.k - 1) kth = dist;
        }
    }
    for (int p = n_valid + lane; p < a.k; p += 64) {
        a.out_ids[qi * a.k + p] = JX_NONE_ID;
        a.out_dist[qi * a.k + p] = __builtin_inff();
    }
    // ---- proof: what was left out is no nearer than the last entry kept, less what the forms can differ by (knn_eps), and
    // that has to exceed the k-th distance.  Comparisons with NaN leave the result unproven
    const uint64_t who = ballot(kth >= 0.f);
    bool proven = n_valid == a.n;
    if (!proven && n_valid == kp + n_odd && odd.count <= KNN_ODD && who) {
        const float e_k = __uint_as_float(readlane32(__float_as_uint(kth), __builtin_ctzll(who)));
        proven = __uint_as_float((uint32_t)(worst >> 32)) - knn_eps(a.d, qq, e_k, __uint_as_float(odd.bb_max), a.parts) > e_k;
    }
    if (lane == 0) a.redo[qi] = proven ? 0u : 1u;
}

// ------------------------------------------------------------------ launch

static int knn_list_regs(int kp) { return kp <= 64 ? 1 : 3; }  // list entries per lane
static bool knn_one_slab(int dtype, int nch) { return dtype == JX_U8 && nch <= 8; }

template <int DT, int NL>
static hipError_t launch_knn(const KnnArgs& a, hipStream_t st) {
    constexpr bool U8 = DT == JX_U8;
    dim3 grid((unsigned)((a.nq + KT - 1) / KT * a.nsplit)), block(256);
    const bool one = knn_one_slab(DT, a.nch);
    if constexpr (U8) {
        if (one) {
            if (a.seed_steps) {
                hipLaunchKernelGGL((knn_u8_kernel<1, true>), grid, block, 0, st, a);
                hipLaunchKernelGGL(knn_limit_kernel, dim3((unsigned)a.nq), dim3(64), 0, st, a);
            }
            hipLaunchKernelGGL((knn_u8_kernel<NL, false>), grid, block, 0, st, a);
        }
    }
    if (!one) {
        const bool few = DT == JX_F32 && a.d <= KNN_FEW_D;
        constexpr bool F32 = DT == JX_F32;
        if (a.seed_steps) {
            if (few) hipLaunchKernelGGL((knn_tile_kernel<DT, 1, true, F32>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((knn_tile_kernel<DT, 1, true>), grid, block, 0, st, a);
            hipLaunchKernelGGL(knn_limit_kernel, dim3((unsigned)a.nq), dim3(64), 0, st, a);
        }
        if (few) hipLaunchKernelGGL((knn_tile_kernel<DT, NL, false, F32>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((knn_tile_kernel<DT, NL, false>), grid, block, 0, st, a);
    }
    hipLaunchKernelGGL((knn_merge_kernel<DT, NL>), dim3((unsigned)a.nq), dim3(64), 0, st, a);
    return hipGetLastError();
}
template <int DT>
static hipError_t launch_knn_lists(const KnnArgs& a, hipStream_t st) {
    return knn_list_regs(a.kp) == 1 ? launch_knn<DT, 1>(a, st) : launch_knn<DT, 3>(a, st);
}

// A few neighbours among vectors of few coordinates: the tiled kernel has as little to do as the vectors are short, this one
// keeps k + KNN_SLACK candidates of float types, a few steps' worth of lists and five launches.  The number of vectors (for
// float types of coordinates) from which this one is at least even; tiled / this in us, d = 16 and k = 1 unless said.
//   float32   1 x 20,000 28.7 / 53.6, 1 x 80,000 55 / 67, 1 x 130,000 93 / 92; 64 x 120,000 252 / 323; 1,000 x 80,000 268 / 463,
//             400 x 160,000 348 / 522, k = 2 1,000 x 640,000 0.93 times as fast; k = 4 1,000 x 260,000 664 / 795, but 100 x
//             160,000 1.13 times as fast; 15,000 x 20,000 0.75, 5,000 x 80,000 even
//   binary16  d = 64 1 x 20,000 36 / 49; 64 x 120,000 287 / 322, 457 x 120,000 350 / 439, 400 x 320,000 1.17 times as fast; k = 4
//             457 x 120,000 355 / 431; from 1,000 queries on ahead
//   uint8     d = 64 1 x 20,000 28.0 / 32.7; 130 x 120,000 249 / 274; 1,000 x 60,000 235 / 258, x 80,000 even
static long long knn_fewest(const BfArgs& b, const long long row) {
    if (b.dtype == JX_U8) {
        if (row >= 96) return 0;
        if (b.nq == 1) return b.k < 4 ? 25000 : 0;
        return b.k > 1 || b.nq <= 48 || b.nq >= 1200 ? 0 : (b.nq < 600 ? 130000 : 70000);
    }
    const bool half = b.dtype == JX_F16;
    long long coords = 0;
    if (b.nq <= 4)
        coords = b.nq * b.k <= (half ? 2 : 0) ? 2000000 : (b.nq * b.k <= 4 ? 1300000 : (b.nq * b.k <= 8 ? 650000 : 0));
    else if (b.nq <= 32)
        coords = 0;
    else if (b.nq <= 64)
        coords = b.k > 1 || row > 128 ? 0 : (half ? 8000000 : 2200000);
    else if (b.nq < (half ? 600 : 2000))
        coords = row > 128 || b.k > 5 ? 0 : (b.k < 4 ? (half ? 10500000 : 5200000) : (half ? 3900000 : (b.nq < 200 ? 1300000 : 4200000)));
    else
        coords = b.k < (half ? 2 : 4) ? 1000000 : 0;
    return coords / b.d;
}

// Takes the search over where it is the faster one and its lists fit scratch_bytes; *done says so.  b.nsplit: the split the
// tiled kernel would run with.
hipError_t launch_knn_tile(const BfArgs& b, void* scratch, long long scratch_bytes, hipStream_t st, char* name, bool* done) {
    *done = false;
    const bool exact = b.dtype == JX_U8;
    const long long row = (long long)b.d * (exact ? 1 : (b.dtype == JX_F16 ? 2 : 4));
    if (((uintptr_t)b.base | (uintptr_t)b.queries) & 15) return hipSuccess;  // rows are read 16 bytes at a time
    if (exact ? row > KU8_ROW : b.d > KNN_FLOAT_D) return hipSuccess;
    KnnArgs a;
    a.base = b.base;
    a.queries = b.queries;
    a.n = b.n;
    a.nq = b.nq;
    a.d = b.d;
    a.nch = (int)(row / 16);
    a.k = b.k;
    a.kp = exact ? b.k : b.k + KNN_SLACK;
    a.parts = b.dtype == JX_F32 ? knn_parts(b.d) : 0.f;
    a.out_ids = b.out_ids;
    a.out_dist = b.out_dist;
    const long long qt = (b.nq + KT - 1) / KT, steps = (b.n + KT - 1) / KT;
    // as many slices as keep every CU at its two workgroups; one workgroup more would be a round of its own
    long long nsplit = KNN_BLOCKS / qt > 1 ? KNN_BLOCKS / qt : 1;
    if (nsplit > steps / 2) nsplit = steps / 2;  // two steps at least
    const long long redo_bytes = (b.nq * 4 + 255) & ~255LL;
    const long long odd_bytes = (qt * (long long)sizeof(KnnOdd) + 255) & ~255LL;
    const long long aux = redo_bytes + odd_bytes + (qt > KNN_BLOCKS ? qt : KNN_BLOCKS) * 16 + 256;
    const long long fit = knn_slices_that_fit(scratch_bytes - aux, b.nq, a.kp);
    if (nsplit > fit) nsplit = fit;
    // Where the tiled kernel stays, tiled / this in us: few vectors (1,000 x 2,000 float32 d = 96, k = 10 181 / 210, 300 x
    // 8,000, k = 1 125 / 155; uint8 300 x 8,000 108 / 111, k = 10 213 / 112); hardly any workgroups; and one neighbour or
    // a few, whose lists cost it little, of more than 64 queries among fewer than 100,000 short vectors (130 x 50,000 uint8,
    // k = 1 176 / 214, but 8,118 x 56,268 1450 / 535, 1,000 x 200,000 615 / 364 and d = 960 1,000 x 20,000 1145 / 669)
    if (nsplit < 1 || qt * nsplit < 64) return hipSuccess;
    if (b.n < (exact ? 6000 : 16384)) return hipSuccess;
    if (b.k < 8 && row < 1024 && b.nq > 64 && b.n < 100000 && b.nq * b.n < 60000000) return hipSuccess;
    if (b.n < knn_fewest(b, row)) return hipSuccess;
    a.nsplit = (int)nsplit;
    a.r_th = (int)((a.kp + nsplit - 1) / nsplit);
    // each slice publishes some more than would make up kp if all were alike, in at most KNN_PUB values
    const int top = a.r_th + (a.r_th < 4 ? a.r_th : 4);
    a.pub_shift = 0;
    while ((top + (1 << a.pub_shift) - 1) >> a.pub_shift > KNN_PUB) a.pub_shift++;
    a.pub = (top + (1 << a.pub_shift) - 1) >> a.pub_shift;
    if (a.pub > KNN_ENTRIES / nsplit) a.pub = (int)(KNN_ENTRIES / nsplit);  // r_th at least: more than 128 slices of kp <= 156
    uint8_t* p = (uint8_t*)scratch + scratch_bytes - aux;  // behind the lists and the published distances
    p -= (uintptr_t)p & 255;
    a.lists = (uint64_t*)scratch;
    a.published = nsplit > 1 ? (uint32_t*)(a.lists + (size_t)b.nq * nsplit * a.kp) : nullptr;
    a.redo = (uint32_t*)p;
    a.odd = (KnnOdd*)(p + redo_bytes);
    a.hopeless = (uint4*)(p + redo_bytes + odd_bytes);  // qt * nsplit <= max(qt, KNN_BLOCKS)
    hipError_t e = hipSuccess;
    // First limits from a share f of every slice.  A tile's 128 queries meet about 128 kp / f vectors below them, each 900
    // cycles of its workgroup (append, its part of a merge, the others waiting); a slab of a step takes 4,000.  The sum of that
    // and of f of the steps is least at f^2 = 28 kp / (steps nslab); a sixteenth at least, a quarter at most.  10,000 x 1M
    // uint8, k = 10, f = 1/16, 1/8, 1/4: 3,452, 3,159, 3,062 us; 1,000 x 100,003 float32 d = 960, k = 100: 1,379, 1,244,
    // 1,172
    const long long each = steps / nsplit;
    const double f = sqrt(28.0 * a.kp / ((double)steps * ((a.nch + 7) / 8)));
    const long long seed = (long long)ceil((double)each * (f < 0.0625 ? 0.0625 : (f > 0.25 ? 0.25 : f)));
    a.seed_steps = a.published && a.r_th <= 32 ? (int)(seed < 1 ? 1 : seed) : 0;
    if (a.published && !a.seed_steps) e = launch_fill_u32(a.published, b.nq * nsplit * a.pub, 0x7F800000u, st);
    if (e != hipSuccess) return e;
    if (!exact && !a.seed_steps) e = launch_fill_u32((uint32_t*)a.odd, qt * (long long)(sizeof(KnnOdd) / 4), 0u, st);
    if (e != hipSuccess) return e;
    *done = true;
    snprintf(name, 96, "knn_tile_kernel<%d,%d,%d> nsplit=%d r_th=%d seed_steps=%d", b.dtype, knn_list_regs(a.kp), knn_one_slab(b.dtype, a.nch) ? 1 : 0, a.nsplit, a.r_th, a.seed_steps);
    if (exact) return launch_knn_lists<JX_U8>(a, st);
    e = b.dtype == JX_F16 ? launch_knn_lists<JX_F16>(a, st) : launch_knn_lists<JX_F32>(a, st);
    if (e != hipSuccess) return e;
    BfArgs again = b;  // tiles with a flagged query, over the lists and the published distances; the caller's split where it fits
    const long long room = (scratch_bytes - aux) / (b.nq * b.k * 8);
    if (again.nsplit > room) again.nsplit = (int)room;
    again.partial = (uint64_t*)scratch;
    again.redo = a.redo;
    return launch_bruteforce(again, st);
}

}  // namespace jx
