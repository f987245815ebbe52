// Rounding rules of the exhaustive search on the matrix cores (knn_tile.hip): plain float arithmetic, so that the test of
// these rules can compile them for the CPU.
#pragma once

#ifdef __HIPCC__
#define JX_HD __host__ __device__ __forceinline__
#else
#define JX_HD inline
#endif

namespace jx {

// What 2 <q, b> is compared with |b|^2 behind, so that every vector whose distance, by either formula of the kernel, is
// below lim passes 2 <q, b> + threshold > |b|^2.  A first threshold counts vectors by |q|^2 - (2 <q, b> - |b|^2) and they
// have to be admitted when the search meets them again.  With u = 2^-24: the two subtractions of the count are off by
// u (|q|^2 + lim) + u lim, the sum here rounds up past |b|^2 <= 2 (|q|^2 + lim) within 4 u (|q|^2 + lim), and the
// operations below lose 3 u (|q|^2 + lim): 9 u in all, and 16 u are added
JX_HD float knn_threshold(float lim, float qq) { return (lim - qq) + (lim + qq) * 0x1p-20f; }

}  // namespace jx
