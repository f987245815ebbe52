// Rounding rules of the exhaustive search on the matrix cores (knn_tile.hip), and how it counts: plain arithmetic, so that the
// test of these rules can compile them for the CPU.
#pragma once
#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define JX_HD __host__ __device__ __forceinline__
#else
#define JX_HD inline
#endif

namespace jx {

#define KT 128  // queries per workgroup, base vectors per step

// What counts base vectors in 32 bits: a set has up to 2^31 - 2 of them, and the step behind the last one begins up to KT - 1
// further on
typedef uint32_t knn_row;
// slice `split` of nsplit; every slice has as many steps, or one more
JX_HD void knn_slice(long long n, int nsplit, int split, knn_row* begin, knn_row* end) {
    const long long steps = (n + KT - 1) / KT, after = (split + 1) * steps / nsplit * KT;
    *begin = (knn_row)(split * steps / nsplit * KT);
    *end = (knn_row)(after > n ? n : after);
}
JX_HD bool knn_whole_step(knn_row b0, knn_row end) { return b0 + KT <= end; }
JX_HD bool knn_last_step(knn_row b0, knn_row end) { return b0 + KT >= end; }

#define KNN_PUB 8  // published distances of one slice and query, at most
// Slices whose lists (kp keys of a query) and published distances have room in so many bytes; a single slice publishes nothing
JX_HD long long knn_slices_that_fit(long long bytes, long long nq, int kp) {
    const long long fit = bytes / (nq * (kp * 8 + KNN_PUB * 4));
    return fit > 0 ? fit : (bytes >= nq * kp * 8 ? 1 : 0);
}

// What 2 <q, b> is compared with |b|^2 behind, so that every vector whose distance, by either formula of the kernel, is
// below lim passes 2 <q, b> + threshold > |b|^2.  A first threshold counts vectors by |q|^2 - (2 <q, b> - |b|^2) and they
// have to be admitted when the search meets them again.  With u = 2^-24: the two subtractions of the count are off by
// u (|q|^2 + lim) + u lim, the sum here rounds up past |b|^2 <= 2 (|q|^2 + lim) within 4 u (|q|^2 + lim), and the
// operations below lose 3 u (|q|^2 + lim): 9 u in all, and 16 u are added
JX_HD float knn_threshold(float lim, float qq) { return (lim - qq) + (lim + qq) * 0x1p-20f; }

// How far the two forms of a vector's distance (the norm form that chooses candidates, the form of the result) can be apart
// if the result's form is at most e: both are sums of d terms, each off by at most (d + 8) 2^-24 (|q| + |b|)^2, the
// comparison with a rounded threshold included, and where squares are subnormal by half of 2^-149 for each of at most 4 d
// operations of the two.  |b| is at most the longest vector's (bb_max = |b|^2, infinity: unknown), and at most |q| + sqrt(e)
// by the triangle inequality, the rounding of e included by the last factor.  Holds up to KNN_FLOAT_D dimensions
#define KNN_FLOAT_D 65536
// parts: what the values of the norm form lack, as a share of (|q| + |b|)^2.  float32 values go to the matrix cores as two
// bfloat16 parts, x = h + l + r.  A bfloat16 has 8 significant bits, so rounding to nearest leaves |l| <= 2^-8 |x| and
// |r| <= 2^-17 |x|, and h h' + h l' + l h' leaves out l l', h r' and r h': at most 2^-15 (1 + 2^-9) |q| |b|, twice that in
// 2 <q, b>, and |q| |b| is at most a quarter of (|q| + |b|)^2: 2^-16 (1 + 2^-9) = 1.53e-5.  A duplicate of a query of
// coordinates 1.0039 comes within 2 % of it.  Where 8 bits leave only 2^-9 and 2^-18 (6e-6, the value here before) the bound
// holds from about 64 dimensions on, by what the first term has to spare.
// An instruction takes 16 coordinates and is off by at most 8 2^-24 of its largest term, subnormals are kept (both measured):
// 3 ceil(d / 16) of them in a row by 24 ceil(d / 16) 2^-24 |q| |b|, in 2 <q, b> at most (0.75 d + 12) 2^-24 (|q| + |b|)^2.  With
// the norms (d / 8 + 7), the sum (4) and the form of the result (d + 2) that is 1.9 d + 25; the first term has 2 d + 32
#define KNN_BF16_PARTS 1.6e-5f
// Up to KNN_FEW_D dimensions a value has three parts (what they leave is nothing) and six products: l r', r l' and r r' are left
// out, 2^-24 (1 + 2^-10) |q| |b|, 2^-25 of the share.  Six instructions are off by 24 where 0.75 d + 12 is spared above: 41.5 of
// 40 at d = 4
#define KNN_FEW_D 16
#define KNN_BF16_THREE 1.5e-7f
JX_HD float knn_parts(int d) { return d <= KNN_FEW_D ? KNN_BF16_THREE : KNN_BF16_PARTS; }  // float32
JX_HD float knn_eps(int d, float qq, float e, float bb_max, float parts = 0.f) {
    const float c = (float)(d + 16) * 1.2e-7f + parts;
    float len = (2.f * sqrtf(qq) + sqrtf(e)) * (1.f + sqrtf(c));
    const float all = sqrtf(qq) + sqrtf(bb_max);
    if (all < len) len = all;
    return c * (len * len) + (float)(d + 16) * 0x1p-147f;  // infinity where a norm of that length could overflow
}

}  // namespace jx
