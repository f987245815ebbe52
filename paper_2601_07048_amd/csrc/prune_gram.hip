// robustPrune (Alg. 3) as a dense contraction, one workgroup per prune.
//
// Whether candidate i discards candidate j (alpha * d(i,j) <= d(p,j), i before j) does not depend on what Alg. 3 has
// selected, so all pair distances of one prune are computed at once from the Gram matrix of its candidate vectors,
//     d(i,j) = G_ii + G_jj - 2 G_ij,   G = X X^T,
// on the matrix cores, and every candidate vector is read exactly once.
//   float32 : rows centred at the pruned vertex p (x_j - x_p: distances are translation invariant and the cancellation
//             in G_ii + G_jj - 2 G_ij then involves local magnitudes only); G_jj is d(p,j) itself.  A centred value of
//             2^-110 and more is the exact sum of three bfloat16 values (8 + 8 + 8 bits of its significand; of smaller ones what
//             lies below 2^-134 is lost, and their squares are zero), and the six products of weight 2^-17 and above go
//             through v_mfma_f32_32x32x16_bf16: 192 cycles for 16 coordinates where v_mfma_f32_32x32x2f32 takes 512.  The
//             second part is at most 2^-8 of a value and the third 2^-17, so the two products of weight 2^-25 and the one
//             behind them are left out, at most 2^-24 (1 + 2^-10) of a product.  Every 32 coordinates have a
//             sum of their own, added to the total by the vector unit, so the result is nearer to the exact one than that
//             of the float32 instruction: relative error of d(i,j) against 64 bits, root mean square / largest,
//             d = 128 1.1e-7 / 4.7e-7 (float32 instruction 2.9e-7 / 1.5e-6), d = 960 1.4e-7 / 5.5e-7 (7.1e-7 / 2.9e-6).
//             Long vectors with alpha above 1 (LONG) take two parts and the three products of them first.  They leave d(i,j) uncertain by 6e-5 of
//             |x_i|^2 + |x_j|^2, which settles all but a few of the 32,000 comparisons of a prune; for those the float32 distance
//             of the two vectors is taken.  Where hundreds are undecided (ties), or squares are subnormal, the three parts are.
//             G_jj is then a float32 sum of the centred values' squares.  Relative error against 64 bits, root mean square /
//             largest, d = 960: those distances 3.7e-8 / 1.1e-7, these sums 4.0e-8 / 1.9e-7.
//   binary16: v_mfma_f32_32x32x16_f16 on the stored values (products exact, float32 accumulation).
//   uint8   : v_mfma_i32_32x32x32_i8 on the values shifted by -128, exact.
//
// The rows are cut into NB blocks of 32, a wavefront each.  Per slab of 128 bytes of every row a wavefront loads, centres
// and splits its own block once and puts it into LDS as MFMA operands; block b then takes the tiles (b, b), (b, b+1), ..
// (b, b + nb/2) modulo nb, which covers every pair of blocks once and gives each wavefront the same number of tiles.  The
// next slab is on its way while one is multiplied.  NB = 4 holds 128 candidates, NB = 8 holds 256.
//
// What bounds it: the matrix cores where vectors are long (d = 960, float32), the relation and the fixpoint where they are
// short.  One wavefront per prune took 450 us for 256 candidates of d = 960, the length of a launch however small its
// batch; a workgroup takes 60.  Build of 20,000 x 960 float32: prunes 62 -> 15 ms, with two parts 11; 60,000 x 128 float32
// 40.6 -> 21.6 ms, binary16 23.9 -> 12.5.
//
// The relation is kept as bit masks by victim, and only with discarders that come before it in (distance, id) order:
// element (i, j) of a tile gives "i discards j" (bits gathered in the lane of j) or "j discards i" (a ballot per row).
// Alg. 3 is then a fixpoint: a candidate with a selected discarder is dead; one whose discarders are all dead is
// selected.  The first undecided candidate in order is always decided, so a round makes progress, and a handful of rounds
// of 40 to 130 instructions replace a walk of up to 256 dependent LDS reads.  Candidates beyond the R-th selected one are
// cut off afterwards: they cannot influence earlier ones.
#include <type_traits>
#include "jx_distance.h"

namespace jx {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef int gi32x16_t __attribute__((ext_vector_type(16)));
typedef int gi32x4_t __attribute__((ext_vector_type(4)));

template <int DT> struct GAcc { typedef f32x16_t type; };
template <> struct GAcc<JX_U8> { typedef gi32x16_t type; };

__device__ __forceinline__ uint4 shift128(uint4 x) {
    x.x ^= 0x80808080u;
    x.y ^= 0x80808080u;
    x.z ^= 0x80808080u;
    x.w ^= 0x80808080u;
    return x;
}
// d(i,j) from G_ii, G_jj (raw bits in the float arrays for uint8) and G_ij, as the float the alpha test uses
template <int DT, typename A>
__device__ __forceinline__ float gram_dist(float ni, float nj, A gij) {
    if constexpr (DT == JX_U8)
        return (float)(uint32_t)(__float_as_int(ni) + __float_as_int(nj) - 2 * (int)gij);
    else
        return fmaxf((ni + nj) - 2.f * (float)gij, 0.f);
}

// two floats -> two bfloat16 (round to nearest even) in one register, and what is left of the floats (exact)
__device__ __forceinline__ uint32_t take_bf16(float& a, float& b) {
    const f32x2_t x = {a, b};
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xFFFF0000u);
    return h;
}

// wavefronts per SIMD that the registers are held to: float32 needs 160 (NB = 4) and 224 of them
#define GT_WAVES(DT, NB) ((DT) != JX_F32 ? 4 : (NB) == 4 ? 3 : 2)
#define GT_SMALL 128
#define GT_BIG 256
// float32: a prune with more undecided pairs takes the three parts on top.  Builds of 12,000 x 960 / 512 with 128 / 256 / 512 /
// 1,024: coordinates of one bit, alpha = 1, 20.5 / 19.4 / 19.4 / 19.4 and 10.8 / 11.0 / 11.4 / 11.5 ms; twelve ones each, alpha = 1,
// 27.7 / 27.9 / 28.7 / 30.5 and 12.8 / 13.0 / 13.6 / 15.7; of normal data, and of all of them with alpha = 1.2, the same
#define GT_PAIRS 256
// two parts: error of G_ij in |x_i| |x_j|.  Roundings to 8 bits leave up to 2^-8 and 2^-16 of a value: 2^-16 for the product of the
// second parts, 2 x 2^-16 (1 + 2^-8) for what is behind them; sums of 32 coordinates and of the slabs, less than (6 + d / 32) 2^-24
#define GT_TWO 6e-5f
#define GT_TINY 1e-28f  // squares below this: products of the parts may be subnormal, and the bound above means nothing
// float32 vectors of so many bytes take two parts first (LONG) where alpha is GT_ALPHA at least.  Builds, three parts / two:
// 20,000 x 960 31.0 / 27.5 ms, 20,000 x 512 17.2 / 16.0, 16,000 x 320 13.25 / 12.8; at 200 dimensions and less 2 % and nothing: the
// relation is the longer part there, and the search for undecided pairs comes on top.  Where distances tie the two parts are made
// in vain.  Coordinates of one bit in clusters, alpha = 1.2: d = 164 9.7 / 10.2 ms, 256 9.7 / 10.0, 320 11.4 / 11.7, 512 11.1 /
// 10.8, 960 19.9 / 17.7.  With alpha = 1 any two candidates as far from each other as from the vertex tie, so copies and
// coordinates of few values do: d = 960 17.3 / 19.4, 512 9.9 / 10.9, copies of every vector 16.1 / 18.3 and 10.3 / 11.1, against
// 18.6 / 17.6 and 11.2 / 11.2 of normal data; with alpha = 1.05 49.3 / 47.9, 10.0 / 9.9, 17.1 / 15.7, 10.9 / 10.6
#define GT_LONG 1280
#define GT_ALPHA 1.05f
#define GT_PIECE 576  // bytes of 32 rows x 16 operand bytes, padded: 64 bytes further on in the banks from piece to piece

template <int DT, int NB>
struct TeamLds {
    static constexpr int M = 32 * NB;
    static constexpr int PIECES = DT == JX_F32 ? 12 : 8;  // operand pieces of a block and slab: [step][part][half]
    union {
        uint8_t slab[NB * PIECES * GT_PIECE];
        struct {
            uint32_t kb[NB * M];   // [w][victim]: which candidates of block w discard the victim
            uint64_t key[M];
            uint32_t by_rank[M];   // slot of the selected candidate of this rank, or JX_NONE_ID
            uint32_t sel_id[M];
            uint32_t sel_dist[M];  // float bits of d(p, selected), selection order
            uint32_t pair[GT_PAIRS];  // float32: pairs that two parts do not decide, discarder << 16 | victim
        };
    };
    uint32_t id[M];
    float dp[M];        // d(p, j); -1 beyond the last candidate: nothing discards it
    float nrm[M];       // G_jj
    uint32_t rank[M];   // place in (distance, id) order
    int pairs;          // entries of pair[], more than GT_PAIRS: all three parts are needed
    int nsel;
};

// Ranks of all candidates where some came without their distance.  All threads of the workgroup.  Ranks and selection are those of
// team_prune and of team_prune_long: as functions of their own the 8-block uint8 merge spills 207 registers for 33, and no deletion
// or insertion of uint8, binary16 or float32 rows takes 1 % longer for it (d = 96 to 960, 72 to 256 candidates).
template <int DT, int NB>
__device__ __forceinline__ void team_ranks(TeamLds<DT, NB>* L, const int m, const int n_fixed, const int tid) {
    if (n_fixed > 0) {
        // ranks: the candidates of known distance are in order already
        uint64_t k = 0;
        if (tid < m) {
            k = ((uint64_t)__float_as_uint(L->dp[tid]) << 32) | L->id[tid];
            L->key[tid] = k;
        }
        __syncthreads();
        if (tid < m) {
            int rank = tid < n_fixed ? 0 : tid - n_fixed;
            for (int t = 0; t < n_fixed; t++) {
                const uint64_t o = L->key[t];
                rank += (o < k || (o == k && t < tid)) ? 1 : 0;
            }
            if (tid < n_fixed) {
                int lo = n_fixed, hi = m;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (L->key[mid] < k) lo = mid + 1;
                    else hi = mid;
                }
                rank += lo - n_fixed;
            }
            L->rank[tid] = (uint32_t)rank;
        }
        __syncthreads();
    }
}

// Alg. 3 on the masks of L->kb, by the first wavefront; the number selected, as team_prune returns it
template <int DT, int NB>
__device__ __forceinline__ int team_select(TeamLds<DT, NB>* L, const int m, const int nb, const bool sorted, const uint32_t p, const int R,
                                           const bool truncated, const int wave, const int lane) {
    using Lds = TeamLds<DT, NB>;
    if (wave == 0) {
        constexpr int H = NB / 2;
        uint32_t kw[H][NB];
        uint64_t U[H], S[H];
#pragma unroll
        for (int h = 0; h < H; h++) {
            const int slot = h * 64 + lane;
            const bool on = slot < m;
#pragma unroll
            for (int w = 0; w < NB; w++) kw[h][w] = on && w < nb && (!sorted || w <= slot >> 5) ? L->kb[w * Lds::M + slot] : 0u;
            U[h] = ballot(on && L->id[on ? slot : 0] != p);
            S[h] = 0;
            L->by_rank[slot] = JX_NONE_ID;
        }
        for (;;) {
            uint64_t any = 0, ns[H], nd[H];
#pragma unroll
            for (int h = 0; h < H; h++) any |= U[h];
            if (!any) break;
#pragma unroll
            for (int h = 0; h < H; h++) {
                uint32_t dead = 0, wait = 0;
#pragma unroll
                for (int w = 0; w < NB; w++) {
                    dead |= kw[h][w] & (uint32_t)(S[w >> 1] >> (32 * (w & 1)));
                    wait |= kw[h][w] & (uint32_t)(U[w >> 1] >> (32 * (w & 1)));
                }
                ns[h] = ballot(dead == 0 && wait == 0) & U[h];
                nd[h] = ballot(dead != 0) & U[h];
            }
#pragma unroll
            for (int h = 0; h < H; h++) {
                U[h] &= ~(ns[h] | nd[h]);
                S[h] |= ns[h];
            }
        }
        wave_sync();
#pragma unroll
        for (int h = 0; h < H; h++)
            if ((S[h] >> lane) & 1ull) L->by_rank[L->rank[h * 64 + lane]] = (uint32_t)(h * 64 + lane);
        wave_sync();
        const int tau = (int)L->rank[m > 0 ? m - 1 : 0];
        int nsel = 0, inside = 0;
#pragma unroll
        for (int h = 0; h < H; h++) {
            const uint32_t slot = L->by_rank[h * 64 + lane];
            const uint64_t on = ballot(slot != JX_NONE_ID);
            const int pos = nsel + prefix_count(on);
            if (slot != JX_NONE_ID && pos < R) {
                L->sel_id[pos] = L->id[slot];
                L->sel_dist[pos] = __float_as_uint(L->dp[slot]);
            }
            nsel += __builtin_popcountll(on);
            inside += __builtin_popcountll(ballot(slot != JX_NONE_ID && h * 64 + lane <= tau));
        }
        // beyond the last candidate of known distance an excluded one could come first
        if (lane == 0) L->nsel = truncated && inside < R ? -1 : (nsel < R ? nsel : R);
    }
    __syncthreads();
    return L->nsel;
}

// L->id[0..m): n_fixed candidates of unknown distance to p, then candidates in ascending (distance, id) order with their
// distances in L->dp.  truncated: further candidates, none before the last one here, exist beyond the pool.  All threads
// of the workgroup call; the arrays are visible (a barrier after they were filled).  Returns the number selected
// (L->sel_id / L->sel_dist, visible to all), or -1 if the pool did not suffice.
template <int DT, int NB>
__device__ __forceinline__ int team_prune(const uint8_t* recs, size_t stride, int vec_bytes, TeamLds<DT, NB>* L, int m, int n_fixed,
                                          uint32_t p, int R, float alpha, bool truncated) {
    using Lds = TeamLds<DT, NB>;
    constexpr int TILES = NB / 2 + 1;
    constexpr int BLOCK = Lds::PIECES * GT_PIECE;
    const int tid = threadIdx.x;
    int lane = lane_id();
    asm volatile("" : "+v"(lane));  // what follows from it is worked out here and not kept across a caller's loop: no registers for that
    const int col = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = (m + 31) >> 5;
    const bool mine = wave < nb;
    if (tid < 32 * nb) {
        L->rank[tid] = tid < m ? (uint32_t)tid : 0xFFFFu;
        if (tid >= m) L->dp[tid] = -1.f;
    }
    typename GAcc<DT>::type acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[t][e] = 0;
    // staging: a load covers 8 rows x 128 bytes
    const int piece = lane & 7, r8 = lane >> 3;
    const uint8_t* rp[4];
    const uint8_t* pp = recs + (size_t)p * stride + piece * 16;
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const int slot = wave * 32 + s * 8 + r8;
        rp[s] = recs + (size_t)(slot < m ? L->id[slot] : p) * stride + piece * 16;
    }
    float fnn[4] = {0.f, 0.f, 0.f, 0.f}, fnp[4] = {0.f, 0.f, 0.f, 0.f}, fpp = 0.f;
    int inn[4] = {0, 0, 0, 0}, inp[4] = {0, 0, 0, 0}, ipp = 0;
    const bool want_dp = DT != JX_F32 && mine && wave * 32 < n_fixed;
    uint8_t* own = L->slab + (size_t)wave * BLOCK;
    uint4 x[4], c;
    auto fetch = [&](int p0) {
        if (p0 + 128 <= vec_bytes) {  // uniform: no lane's load waits for a branch
            c = load16(pp + p0);
#pragma unroll
            for (int s = 0; s < 4; s++) x[s] = load16(rp[s] + p0);
            if constexpr (DT == JX_U8) {
                c = shift128(c);
#pragma unroll
                for (int s = 0; s < 4; s++) x[s] = shift128(x[s]);
            }
        } else {  // the last piece of a row: zeros (after the shift) beyond the data
            const bool in = p0 + piece * 16 < vec_bytes;
            const uint4 zero = make_uint4(0, 0, 0, 0);
            c = in ? load16(pp + p0) : zero;
#pragma unroll
            for (int s = 0; s < 4; s++) x[s] = in ? load16(rp[s] + p0) : zero;
            if (DT == JX_U8 && in) {
                c = shift128(c);
#pragma unroll
                for (int s = 0; s < 4; s++) x[s] = shift128(x[s]);
            }
        }
    };
    if (mine) fetch(0);
    for (int p0 = 0; p0 < vec_bytes; p0 += 128) {
        if (mine) {
            if constexpr (DT == JX_F32) {
                uint8_t* at = own + (((piece >> 2) * 6 + ((piece >> 1) & 1)) * GT_PIECE) + (piece & 1) * 8 + r8 * 16;
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    float v0 = __uint_as_float(x[s].x) - __uint_as_float(c.x), v1 = __uint_as_float(x[s].y) - __uint_as_float(c.y);
                    float v2 = __uint_as_float(x[s].z) - __uint_as_float(c.z), v3 = __uint_as_float(x[s].w) - __uint_as_float(c.w);
#pragma unroll
                    for (int part = 0; part < 3; part++) {
                        uint2 h;
                        h.x = take_bf16(v0, v1);
                        h.y = take_bf16(v2, v3);
                        *reinterpret_cast<uint2*>(at + part * 2 * GT_PIECE + s * 128) = h;
                    }
                }
            } else {
#pragma unroll
                for (int s = 0; s < 4; s++) *reinterpret_cast<uint4*>(own + piece * GT_PIECE + (s * 8 + r8) * 16) = x[s];
                if (want_dp) {
                    if constexpr (DT == JX_F16) {
                        fpp = hdot2(c.w, c.w, hdot2(c.z, c.z, hdot2(c.y, c.y, hdot2(c.x, c.x, fpp))));
#pragma unroll
                        for (int s = 0; s < 4; s++) {
                            fnn[s] = hdot2(x[s].w, x[s].w, hdot2(x[s].z, x[s].z, hdot2(x[s].y, x[s].y, hdot2(x[s].x, x[s].x, fnn[s]))));
                            fnp[s] = hdot2(x[s].w, c.w, hdot2(x[s].z, c.z, hdot2(x[s].y, c.y, hdot2(x[s].x, c.x, fnp[s]))));
                        }
                    } else {
                        auto dot = [](const uint4& a, const uint4& b, int t) {
                            t = __builtin_amdgcn_sdot4((int)a.x, (int)b.x, t, false);
                            t = __builtin_amdgcn_sdot4((int)a.y, (int)b.y, t, false);
                            t = __builtin_amdgcn_sdot4((int)a.z, (int)b.z, t, false);
                            return __builtin_amdgcn_sdot4((int)a.w, (int)b.w, t, false);
                        };
                        ipp = dot(c, c, ipp);
#pragma unroll
                        for (int s = 0; s < 4; s++) {
                            inn[s] = dot(x[s], x[s], inn[s]);
                            inp[s] = dot(x[s], c, inp[s]);
                        }
                    }
                }
            }
            if (p0 + 128 < vec_bytes) fetch(p0 + 128);
        }
        __syncthreads();
        if (mine) {
            const uint8_t* opnd = L->slab + half * GT_PIECE + col * 16;
            if constexpr (DT == JX_F32) {
                bf16x8_t a[2][3];
#pragma unroll
                for (int q = 0; q < 6; q++)
                    a[q / 3][q % 3] = *reinterpret_cast<const bf16x8_t*>(opnd + (size_t)wave * BLOCK + q * 2 * GT_PIECE);
#pragma unroll
                for (int t = 0; t < TILES; t++) {
                    if (2 * t < nb || t == 0 || (2 * t == nb && wave < t)) {  // uniform
                        const int bj = wave + t < nb ? wave + t : wave + t - nb;
                        // a sum of its own for the 32 coordinates of the slab, the smallest products first
                        f32x16_t part;
#pragma unroll
                        for (int e = 0; e < 16; e++) part[e] = 0.f;
#pragma unroll
                        for (int ks = 0; ks < 2; ks++) {
                            bf16x8_t b[3];
#pragma unroll
                            for (int q = 0; q < 3; q++)
                                b[q] = *reinterpret_cast<const bf16x8_t*>(opnd + (size_t)bj * BLOCK + (ks * 3 + q) * 2 * GT_PIECE);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][2], b[0], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[2], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][1], b[1], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][1], b[0], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[1], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[0], part, 0, 0, 0);
                        }
#pragma unroll
                        for (int e = 0; e < 16; e++) acc[t][e] += part[e];
                    }
                }
            } else {
#pragma unroll
                for (int ks = 0; ks < 4; ks++) {
                    const uint4 a = *reinterpret_cast<const uint4*>(opnd + (size_t)wave * BLOCK + ks * 2 * GT_PIECE);
#pragma unroll
                    for (int t = 0; t < TILES; t++) {
                        if (2 * t < nb || t == 0 || (2 * t == nb && wave < t)) {  // uniform
                            const int bj = wave + t < nb ? wave + t : wave + t - nb;
                            const uint4 b = *reinterpret_cast<const uint4*>(opnd + (size_t)bj * BLOCK + ks * 2 * GT_PIECE);
                            if constexpr (DT == JX_U8)
                                acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(gi32x4_t, a), __builtin_bit_cast(gi32x4_t, b),
                                                                               acc[t], 0, 0, 0);
                            else
                                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b),
                                                                                acc[t], 0, 0, 0);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    // Accumulator layout of the 32x32 tiles: register e of lane (col, half) holds row 8*(e/4) + 4*half + e%4, column col.
    // ---- G_jj from the diagonal tiles, d(p, j) of the candidates that came without
    if (mine) {
        const int hcol = (col >> 2) & 1, ecol = ((col >> 3) << 2) | (col & 3);
        float dv = 0.f;
#pragma unroll
        for (int e = 0; e < 16; e++)
            if (e == ecol) {
                if constexpr (DT == JX_U8)
                    dv = __int_as_float(acc[0][e]);
                else
                    dv = acc[0][e];
            }
        if (half == hcol) {
            L->nrm[wave * 32 + col] = dv;
            if (DT == JX_F32 && wave * 32 + col < n_fixed) {
                if (dv != dv) {  // a square overflowed, or a value is not finite: products of the parts have both signs
                    dv = 0.f;
                    const float* xr = reinterpret_cast<const float*>(recs + (size_t)L->id[wave * 32 + col] * stride);
                    const float* pr = reinterpret_cast<const float*>(recs + (size_t)p * stride);
#pragma unroll 1
                    for (int e = 0; e < vec_bytes / 4; e++) dv = fmaf(xr[e] - pr[e], xr[e] - pr[e], dv);
                }
                L->dp[wave * 32 + col] = dv;
            }
        }
        if (want_dp) {
            if constexpr (DT == JX_F16) fpp = group_sum<8>(fpp);
            if constexpr (DT == JX_U8) ipp = group_sum<8>(ipp);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                float d = 0.f;
                if constexpr (DT == JX_F16) d = fmaxf((fpp + group_sum<8>(fnn[s])) - 2.f * group_sum<8>(fnp[s]), 0.f);
                if constexpr (DT == JX_U8) d = (float)(uint32_t)(ipp + group_sum<8>(inn[s]) - 2 * group_sum<8>(inp[s]));
                const int slot = wave * 32 + s * 8 + r8;
                if (piece == 0 && slot < n_fixed) L->dp[slot] = d;
            }
        }
    }
    __syncthreads();
    team_ranks<DT, NB>(L, m, n_fixed, tid);
    // ---- the discard relation, tile by tile.  Candidates that came in order (n_fixed = 0) are discarded by those of their own
    // block and of blocks before it only: half of it
    const bool sorted = n_fixed == 0;
    if (mine) {
#pragma unroll
        for (int t = 0; t < TILES; t++) {
            if (2 * t < nb || t == 0 || (2 * t == nb && wave < t)) {  // uniform
                const int bj = wave + t < nb ? wave + t : wave + t - nb;
                const int j = bj * 32 + col;
                const float nj = L->nrm[j], dpj = L->dp[j];
                const uint32_t rj = L->rank[j];
                const bool fwd = !sorted || wave <= bj, back = t > 0 && (!sorted || bj < wave);
                uint32_t victim_j = 0, victim_i = 0;
                if (fwd) {
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const int i0 = wave * 32 + 8 * g + 4 * half;
                        const float4 n4 = *reinterpret_cast<const float4*>(&L->nrm[i0]);
                        const uint4 r4 = *reinterpret_cast<const uint4*>(&L->rank[i0]);
                        const float ni[4] = {n4.x, n4.y, n4.z, n4.w};
                        const uint32_t ri[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
                        for (int f = 0; f < 4; f++) {
                            const float ad = __fmul_rn(alpha, gram_dist<DT>(ni[f], nj, acc[t][4 * g + f]));
                            if (ri[f] < rj && ad <= dpj) victim_j |= 1u << (8 * g + f);
                        }
                    }
                    victim_j <<= 4 * half;
                    victim_j |= shfl_xor(victim_j, 32);
                    if (half == 0) L->kb[wave * Lds::M + j] = victim_j;
                }
                if (back) {
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const int i0 = wave * 32 + 8 * g + 4 * half;
                        const float4 n4 = *reinterpret_cast<const float4*>(&L->nrm[i0]);
                        const float4 d4 = *reinterpret_cast<const float4*>(&L->dp[i0]);
                        const uint4 r4 = *reinterpret_cast<const uint4*>(&L->rank[i0]);
                        const float ni[4] = {n4.x, n4.y, n4.z, n4.w}, di[4] = {d4.x, d4.y, d4.z, d4.w};
                        const uint32_t ri[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
                        for (int f = 0; f < 4; f++) {
                            const float ad = __fmul_rn(alpha, gram_dist<DT>(ni[f], nj, acc[t][4 * g + f]));
                            const uint64_t mi = ballot(rj < ri[f] && ad <= di[f]);
                            const uint32_t row = (col & 4) ? (uint32_t)(mi >> 32) : (uint32_t)mi;  // of the lane's own row, if it is among these two
                            if (4 * g + f == (((col >> 3) << 2) | (col & 3))) victim_i = row;
                        }
                    }
                    if (half == 0) L->kb[bj * Lds::M + wave * 32 + col] = victim_i;
                }
            }
        }
    }
    __syncthreads();
    return team_select<DT, NB>(L, m, nb, sorted, p, R, truncated, wave, lane);
}

// team_prune for long float32 vectors: two parts first (see above).
template <int NB>
__device__ __forceinline__ int team_prune_long(const uint8_t* recs, size_t stride, int vec_bytes, TeamLds<JX_F32, NB>* L, int m, int n_fixed,
                                          uint32_t p, int R, float alpha, bool truncated) {
    constexpr int DT = JX_F32;
    using Lds = TeamLds<DT, NB>;
    constexpr int TILES = NB / 2 + 1;
    constexpr int BLOCK = Lds::PIECES * GT_PIECE;
    const int tid = threadIdx.x;
    int lane = lane_id();
    asm volatile("" : "+v"(lane));  // what follows from it is worked out here and not kept across a caller's loop: no registers for that
    const int col = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = (m + 31) >> 5;
    const bool mine = wave < nb;
    if (tid < 32 * nb) {
        L->rank[tid] = tid < m ? (uint32_t)tid : 0xFFFFu;
        if (tid >= m) L->dp[tid] = -1.f;
    }
    typename GAcc<DT>::type acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[t][e] = 0;
    // staging: a load covers 8 rows x 128 bytes
    const int piece = lane & 7, r8 = lane >> 3;
    const uint8_t* rp[4];
    const uint8_t* pp = recs + (size_t)p * stride + piece * 16;
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const int slot = wave * 32 + s * 8 + r8;
        rp[s] = recs + (size_t)(slot < m ? L->id[slot] : p) * stride + piece * 16;
    }
    float fnn[4] = {0.f, 0.f, 0.f, 0.f};
    uint8_t* own = L->slab + (size_t)wave * BLOCK;
    uint4 x[4], c;
    auto fetch = [&](int p0) {
        if (p0 + 128 <= vec_bytes) {  // uniform: no lane's load waits for a branch
            c = load16(pp + p0);
#pragma unroll
            for (int s = 0; s < 4; s++) x[s] = load16(rp[s] + p0);
        } else {  // the last piece of a row: zeros (after the shift) beyond the data
            const bool in = p0 + piece * 16 < vec_bytes;
            const uint4 zero = make_uint4(0, 0, 0, 0);
            c = in ? load16(pp + p0) : zero;
#pragma unroll
            for (int s = 0; s < 4; s++) x[s] = in ? load16(rp[s] + p0) : zero;
        }
    };
    auto gram = [&](auto parts) __attribute__((always_inline)) {
    constexpr int PARTS = decltype(parts)::value;
    if (mine) fetch(0);
    for (int p0 = 0; p0 < vec_bytes; p0 += 128) {
        if (mine) {
            {
                uint8_t* at = own + (((piece >> 2) * (2 * PARTS) + ((piece >> 1) & 1)) * GT_PIECE) + (piece & 1) * 8 + r8 * 16;
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    float v0 = __uint_as_float(x[s].x) - __uint_as_float(c.x), v1 = __uint_as_float(x[s].y) - __uint_as_float(c.y);
                    float v2 = __uint_as_float(x[s].z) - __uint_as_float(c.z), v3 = __uint_as_float(x[s].w) - __uint_as_float(c.w);
                    if (PARTS == 2) fnn[s] += fmaf(v3, v3, fmaf(v2, v2, fmaf(v1, v1, v0 * v0)));
#pragma unroll
                    for (int part = 0; part < PARTS; part++) {
                        uint2 h;
                        h.x = take_bf16(v0, v1);
                        h.y = take_bf16(v2, v3);
                        *reinterpret_cast<uint2*>(at + part * 2 * GT_PIECE + s * 128) = h;
                    }
                }
            }
            if (p0 + 128 < vec_bytes) fetch(p0 + 128);
        }
        __syncthreads();
        if (mine) {
            const uint8_t* opnd = L->slab + half * GT_PIECE + col * 16;
            {
                bf16x8_t a[2][PARTS];
#pragma unroll
                for (int q = 0; q < 2 * PARTS; q++)
                    a[q / PARTS][q % PARTS] = *reinterpret_cast<const bf16x8_t*>(opnd + (size_t)wave * BLOCK + q * 2 * GT_PIECE);
#pragma unroll
                for (int t = 0; t < TILES; t++) {
                    if (2 * t < nb || t == 0 || (2 * t == nb && wave < t)) {  // uniform
                        const int bj = wave + t < nb ? wave + t : wave + t - nb;
                        // a sum of its own for the 32 coordinates of the slab, the smallest products first
                        f32x16_t part;
#pragma unroll
                        for (int e = 0; e < 16; e++) part[e] = 0.f;
#pragma unroll
                        for (int ks = 0; ks < 2; ks++) {
                            bf16x8_t b[PARTS];
#pragma unroll
                            for (int q = 0; q < PARTS; q++)
                                b[q] = *reinterpret_cast<const bf16x8_t*>(opnd + (size_t)bj * BLOCK + (ks * PARTS + q) * 2 * GT_PIECE);
                            if constexpr (PARTS == 3) {
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][2], b[0], part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[2], part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][1], b[1], part, 0, 0, 0);
                            }
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][1], b[0], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[1], part, 0, 0, 0);
                            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[0], part, 0, 0, 0);
                        }
#pragma unroll
                        for (int e = 0; e < 16; e++) acc[t][e] += part[e];
                    }
                }
            }
        }
        __syncthreads();
    }
    };
    gram(std::integral_constant<int, 2>());
    // Accumulator layout of the 32x32 tiles: register e of lane (col, half) holds row 8*(e/4) + 4*half + e%4, column col.
    // ---- G_jj from the diagonal tiles (float32: the sums of the centred values' squares), d(p, j) of the candidates that came without
    if (tid == 0) L->pairs = 0;
    if (mine) {
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const float n = group_sum<8>(fnn[s]);
            const int slot = wave * 32 + s * 8 + r8;
            if (piece == 0) {
                L->nrm[slot] = n;
                if (slot < n_fixed) L->dp[slot] = n;
            }
        }
    }
    __syncthreads();
    team_ranks<DT, NB>(L, m, n_fixed, tid);
    // ---- the discard relation, tile by tile.  Candidates that came in order (n_fixed = 0) are discarded by those of their own
    // block and of blocks before it only: half of it
    const bool sorted = n_fixed == 0;
    if (tid < m && L->nrm[tid] > 0.f && L->nrm[tid] < GT_TINY) L->pairs = GT_PAIRS + 1;
    const float two = GT_TWO * 1.01f * alpha;
    // undecided: |alpha d(i,j) - d(p,j)| within alpha times the error of d(i,j), 2 GT_TWO |x_i| |x_j| at most.  An infinite d(p,j)
    // is decided.  The slots behind the last candidate have no vector to read: a vector with an infinite coordinate is undecided
    // against each of them (its norm is infinite, its product with a row of zeros is NaN and its distance 0 for it)
    auto list = [&](const typename GAcc<DT>::type& g, const float nj, const int j, const float dpj, const uint32_t rj, const bool j_first) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int i = wave * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
            const float ni = L->nrm[i], dv = j_first ? L->dp[i] : dpj;
            const uint32_t ri = L->rank[i];
            if ((j_first ? rj < ri : ri < rj) && (j_first ? i : j) < m && fmaf(-two, ni + nj, fabsf(__fmul_rn(alpha, gram_dist<DT>(ni, nj, g[e])) - dv)) < 0.f) {
                const int at = atomicAdd(&L->pairs, 1);
                if (at < GT_PAIRS) L->pair[at] = j_first ? (uint32_t)(j << 16 | i) : (uint32_t)(i << 16 | j);
            }
        }
    };
    auto relate = [&](const bool mark) __attribute__((always_inline)) {
    if (mine) {
#pragma unroll
        for (int t = 0; t < TILES; t++) {
            if (2 * t < nb || t == 0 || (2 * t == nb && wave < t)) {  // uniform
                const int bj = wave + t < nb ? wave + t : wave + t - nb;
                const int j = bj * 32 + col;
                const float nj = L->nrm[j], dpj = L->dp[j];
                const uint32_t rj = L->rank[j];
                const bool fwd = !sorted || wave <= bj, back = t > 0 && (!sorted || bj < wave);
                uint32_t victim_j = 0, victim_i = 0;
                if (fwd) {
                    float near = 0.f;
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const int i0 = wave * 32 + 8 * g + 4 * half;
                        const float4 n4 = *reinterpret_cast<const float4*>(&L->nrm[i0]);
                        const uint4 r4 = *reinterpret_cast<const uint4*>(&L->rank[i0]);
                        const float ni[4] = {n4.x, n4.y, n4.z, n4.w};
                        const uint32_t ri[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
                        for (int f = 0; f < 4; f++) {
                            const float ad = __fmul_rn(alpha, gram_dist<DT>(ni[f], nj, acc[t][4 * g + f]));
                            if (ri[f] < rj && ad <= dpj) victim_j |= 1u << (8 * g + f);
                            if (mark) near = fminf(near, fmaf(-two, ni[f] + nj, fabsf(ad - dpj)));
                        }
                    }
                    if (mark && ballot(near < 0.f)) list(acc[t], nj, j, dpj, rj, false);
                    victim_j <<= 4 * half;
                    victim_j |= shfl_xor(victim_j, 32);
                    if (half == 0) L->kb[wave * Lds::M + j] = victim_j;
                }
                if (back) {
                    float near = 0.f;
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const int i0 = wave * 32 + 8 * g + 4 * half;
                        const float4 n4 = *reinterpret_cast<const float4*>(&L->nrm[i0]);
                        const float4 d4 = *reinterpret_cast<const float4*>(&L->dp[i0]);
                        const uint4 r4 = *reinterpret_cast<const uint4*>(&L->rank[i0]);
                        const float ni[4] = {n4.x, n4.y, n4.z, n4.w}, di[4] = {d4.x, d4.y, d4.z, d4.w};
                        const uint32_t ri[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
                        for (int f = 0; f < 4; f++) {
                            const float ad = __fmul_rn(alpha, gram_dist<DT>(ni[f], nj, acc[t][4 * g + f]));
                            const uint64_t mi = ballot(rj < ri[f] && ad <= di[f]);
                            if (mark) near = fminf(near, fmaf(-two, ni[f] + nj, fabsf(ad - di[f])));
                            const uint32_t row = (col & 4) ? (uint32_t)(mi >> 32) : (uint32_t)mi;  // of the lane's own row, if it is among these two
                            if (4 * g + f == (((col >> 3) << 2) | (col & 3))) victim_i = row;
                        }
                    }
                    if (mark && ballot(near < 0.f)) list(acc[t], nj, j, dpj, rj, true);
                    if (half == 0) L->kb[bj * Lds::M + wave * 32 + col] = victim_i;
                }
            }
        }
    }
    };
    relate(true);
    __syncthreads();
    const int pairs = L->pairs;
    if (pairs > GT_PAIRS) {  // ties by the hundred, or squares too small: the products of three parts
        __syncthreads();
#pragma unroll
        for (int t = 0; t < TILES; t++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[t][e] = 0;
        gram(std::integral_constant<int, 3>());
        relate(false);
    } else {
        for (int k = wave; k < pairs; k += NB) {  // a wavefront per pair: the float32 distance of the vectors
            const uint32_t ij = L->pair[k];
            const int i = (int)(ij >> 16), j = (int)(ij & 0xFFFFu);
            const float* xi = reinterpret_cast<const float*>(recs + (size_t)L->id[i] * stride);
            const float* xj = reinterpret_cast<const float*>(recs + (size_t)L->id[j] * stride);
            float d = 0.f;
            for (int e = lane * 4; e < vec_bytes / 4; e += 256) {
                const float4 u = *reinterpret_cast<const float4*>(xi + e), w = *reinterpret_cast<const float4*>(xj + e);
                d += fmaf(u.w - w.w, u.w - w.w, fmaf(u.z - w.z, u.z - w.z, fmaf(u.y - w.y, u.y - w.y, (u.x - w.x) * (u.x - w.x))));
            }
            d = group_sum<64>(d);
            uint32_t* word = &L->kb[(i >> 5) * Lds::M + j];
            if (lane == 0) {
                if (__fmul_rn(alpha, d) <= L->dp[j]) atomicOr(word, 1u << (i & 31));
                else atomicAnd(word, ~(1u << (i & 31)));
            }
        }
    }
    __syncthreads();
    return team_select<DT, NB>(L, m, nb, sorted, p, R, truncated, wave, lane);
}

// ---- forward prune of the candidate list of each new point (Alg. 4 step 2): lists of at most 128 (NB = 4), or of 129 to
// 256 and the closest 256 of a longer one (NB = 8; exact if Alg. 3 finds R neighbours in them).  NB = 8 marks every point
// of the batch in a.dead[i * a.L]: 0xFF = row and reverse edges written here, 0 = left to the list-based kernel (which
// leaves lists of at most 128 alone).
template <int DT, int NB, bool LONG>
__global__ void __launch_bounds__(NB * 64, GT_WAVES(DT, NB)) forward_prune_gram_kernel(InsertArgs a) {
    __shared__ TeamLds<DT, NB> lds;
    TeamLds<DT, NB>* L = &lds;
    const int tid = threadIdx.x, lane = lane_id();
    const long long i = a.first + blockIdx.x;
    long long xid = a.id_base + i;
    if (xid >= a.id_skip) xid++;
    const uint32_t* ids = a.cand_ids + (size_t)i * a.L;
    const uint32_t* dbits = a.cand_dist + (size_t)i * a.L;
    int nB = 0;
    for (int c0 = 0; c0 < a.L; c0 += 64) {
        const int j = c0 + lane;
        const bool valid = j < a.L && ids[j] != JX_NONE_ID;  // the list is filled from the left
        nB += __builtin_popcountll(ballot(valid));
    }
    if (NB == 8 && nB <= GT_SMALL && tid == 0) a.dead[(size_t)i * a.L] = 0;
    if ((NB == 8) != (nB > GT_SMALL)) return;
    const int m = nB < 32 * NB ? nB : 32 * NB;
    for (int j = tid; j < m; j += NB * 64) {
        L->id[j] = ids[j];
        L->dp[j] = __uint_as_float(dbits[j]);
    }
    __syncthreads();
    int nsel;
    if constexpr (LONG) nsel = team_prune_long<NB>(a.ds.recs, (size_t)a.ds.rec_stride, a.ds.nch * 16, L, m, 0, (uint32_t)xid, a.R, a.alpha, m < nB);
    else nsel = team_prune<DT, NB>(a.ds.recs, (size_t)a.ds.rec_stride, a.ds.nch * 16, L, m, 0, (uint32_t)xid, a.R, a.alpha, m < nB);
    if (NB == 8 && tid == 0) a.dead[(size_t)i * a.L] = nsel < 0 ? 0 : 0xFF;
    if (nsel < 0) return;
    if (DT == JX_U8 && tid == 0) a.clean[xid] = (uint8_t)(nsel < 255 ? nsel : 255);
    uint32_t* row = a.adj + (size_t)xid * a.R;
    for (int j = tid; j < a.R; j += NB * 64) {
        const bool on = j < nsel;
        const uint32_t v = on ? L->sel_id[j] : JX_NONE_ID;
        row[j] = v;
        a.keys[(size_t)i * a.R + j] = on ? (((uint64_t)v << 32) | L->sel_dist[j]) : JX_EMPTY_KEY;
        a.vals[(size_t)i * a.R + j] = on ? (uint32_t)xid : JX_NONE_ID;
    }
}

// ---- reverse-edge merge (Alg. 4 step 3)
// A thread per segment: appends where the row still fits, and lists the others by size, so that no workgroup of the
// kernels below spends a chain of dependent loads on a segment that is not its own.  An entry holds the segment, the
// degree of its row and the number of new edges (at most 4,095 are told apart); lists[0..) is the list of the small
// ones (at most small_max candidates), lists[.. E - 1] downwards that of the large ones; rows of more than deg_max
// neighbours leave a large one too little room for new edges.  fresh[0..) (or NULL) is the list of the rows whose first
// entries one prune selected, with at most FRESH_MAX others (prune_u8.hip).
__global__ void __launch_bounds__(256) reverse_class_kernel(InsertArgs a, int small_max, int deg_max) {
    const int lane = lane_id();
    const long long nseg = *a.nseg;
    const long long total = a.E ? a.E : a.B * a.R;
    for (long long s0 = (long long)blockIdx.x * 256; s0 < nseg; s0 += (long long)gridDim.x * 256) {
        const long long s = s0 + threadIdx.x;
        int cls = 0;
        uint64_t entry = 0;
        const uint32_t head = s < nseg ? a.heads[s] : 0x80000000u;
        if (!(head & 0x80000000u)) {  // not done by a kernel before
            const long long lo = head;
            const uint32_t v = (uint32_t)(a.keys[lo] >> 32);
            long long known = 1, step = 1;  // keys[lo .. lo + known) belong to v
            while (lo + known + step - 1 < total && (uint32_t)(a.keys[lo + known + step - 1] >> 32) == v) {
                known += step;
                step *= 2;
            }
            long long end = known + step - 1 < total - lo ? known + step - 1 : total - lo;
            while (known < end) {
                const long long mid = (known + end) >> 1;
                if ((uint32_t)(a.keys[lo + mid] >> 32) == v) known = mid + 1;
                else end = mid;
            }
            const long long m = known;
            uint32_t* row = a.adj + (size_t)v * a.R;
            int deg = 0;
            if (!a.force_prune) {
                int hi = a.R;
                while (deg < hi) {  // the row is filled from the left
                    const int mid = (deg + hi) >> 1;
                    if (row[mid] != JX_NONE_ID) deg = mid + 1;
                    else hi = mid;
                }
            }
            if (!a.force_prune && deg + m <= a.R) {
                for (int j = 0; j < (int)m; j++) row[deg + j] = a.vals[lo + j];
                const_cast<uint32_t*>(a.heads)[s] = (uint32_t)lo | 0x80000000u;
            } else {
                cls = deg + m <= small_max ? 1 : (deg <= deg_max ? 2 : 0);
                if (a.fresh) {
                    const int c = a.clean[v];
                    if (c > 0 && c <= 64 && c <= deg && deg - c + m <= FRESH_MAX && deg + m > 32) cls = 3;
                }
                entry = (uint64_t)s | ((uint64_t)((uint32_t)deg << 12 | (uint32_t)(m < 4095 ? m : 4095)) << 32);
            }
        }
#pragma unroll
        for (int k = 1; k <= 3; k++) {
            const uint64_t on = ballot(cls == k);
            if (!on) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(const_cast<uint32_t*>(a.nseg) + k, (uint32_t)__builtin_popcountll(on));
            at = readlane32(at, 0) + (uint32_t)prefix_count(on);
            if (cls == k && k == 3) a.fresh[at] = (uint32_t)s;
            else if (cls == k) a.lists[k == 1 ? (long long)at : total - 1 - at] = entry;
        }
    }
}

// NB = 4: at most 128 candidates.  NB = 8: up to 256, or the existing neighbours and the closest new edges up to 256 (the
// new edges arrive sorted); a pool that does not yield R neighbours no farther than its last new edge is left to the
// list-based kernel.  A segment that is done is marked (bit 31 of its head): its rewritten row no longer tells.
template <int DT, int NB, bool LONG>
__global__ void __launch_bounds__(NB * 64, GT_WAVES(DT, NB)) reverse_merge_gram_kernel(InsertArgs a) {
    __shared__ TeamLds<DT, NB> lds;
    TeamLds<DT, NB>* L = &lds;
    const int tid = threadIdx.x;
    const uint32_t n = a.nseg[NB == 4 ? 1 : 2];
    const long long total = a.E ? a.E : a.B * a.R;
    for (uint32_t at = blockIdx.x; at < n; at += gridDim.x) {
        const uint64_t entry = a.lists[NB == 4 ? (long long)at : total - 1 - at];
        const uint32_t s = (uint32_t)entry;
        const int deg = seg_deg(entry), m = seg_new(entry);
        const long long lo = a.heads[s];
        const uint32_t v = (uint32_t)(a.keys[lo] >> 32);
        uint32_t* row = a.adj + (size_t)v * a.R;
        const int mp = m < 32 * NB - deg ? m : 32 * NB - deg;
        for (int j = tid; j < deg; j += NB * 64) L->id[j] = row[j];
        for (int j = tid; j < mp; j += NB * 64) {
            L->id[deg + j] = a.vals[lo + j];
            L->dp[deg + j] = __uint_as_float((uint32_t)a.keys[lo + j]);
        }
        __syncthreads();
        int nsel;
        if constexpr (LONG) nsel = team_prune_long<NB>(a.ds.recs, (size_t)a.ds.rec_stride, a.ds.nch * 16, L, deg + mp, deg, v, a.R, a.alpha, mp < m);
        else nsel = team_prune<DT, NB>(a.ds.recs, (size_t)a.ds.rec_stride, a.ds.nch * 16, L, deg + mp, deg, v, a.R, a.alpha, mp < m);
        if (nsel >= 0) {
            for (int j = tid; j < a.R; j += NB * 64) row[j] = j < nsel ? L->sel_id[j] : JX_NONE_ID;
            if (DT == JX_U8 && tid == 0) a.clean[v] = (uint8_t)(nsel < 255 ? nsel : 255);
            if (tid == 0) const_cast<uint32_t*>(a.heads)[s] = (uint32_t)lo | 0x80000000u;
        }
        __syncthreads();
    }
}

hipError_t launch_reverse_class(const InsertArgs& a, int small_max, int deg_max, hipStream_t st) {
    const long long want = ((a.E ? a.E : a.B * a.R) + 255) / 256;
    hipLaunchKernelGGL(reverse_class_kernel, dim3((unsigned)(want < 1024 ? (want < 1 ? 1 : want) : 1024)), dim3(256), 0, st, a, small_max, deg_max);
    return hipGetLastError();
}

template <int DT, bool LONG = false>
static hipError_t launch_forward_gram_dt(const InsertArgs& a, hipStream_t st) {
    constexpr long long MOST = 1 << 22;  // workgroups of a launch, which has fewer than 2^32 threads
    for (InsertArgs s = a; s.first < a.B; s.first += MOST) {
        const dim3 grid((unsigned)(a.B - s.first < MOST ? a.B - s.first : MOST));
        hipLaunchKernelGGL((forward_prune_gram_kernel<DT, 4, LONG>), grid, dim3(256), 0, st, s);
        if (a.L > GT_SMALL) hipLaunchKernelGGL((forward_prune_gram_kernel<DT, 8, LONG>), grid, dim3(512), 0, st, s);
    }
    return hipGetLastError();
}

template <int DT, bool LONG = false>
static hipError_t launch_reverse_gram_dt(const InsertArgs& a, hipStream_t st) {
    const long long most = a.E ? a.E : a.B * a.R;  // segments there can be
    auto grid = [&](long long cap) { return dim3((unsigned)(most < cap ? (most < 1 ? 1 : most) : cap)); };
    hipError_t e = launch_reverse_class(a, GT_SMALL, GT_BIG - 64, st);
    if (e != hipSuccess) return e;
    // persistent workgroups: as many as the card holds, twice over
    hipLaunchKernelGGL((reverse_merge_gram_kernel<DT, 4, LONG>), grid(2048), dim3(256), 0, st, a);
    if (segment_most(a) > GT_SMALL) hipLaunchKernelGGL((reverse_merge_gram_kernel<DT, 8, LONG>), grid(1024), dim3(512), 0, st, a);
    return hipGetLastError();
}

static bool two_parts_first(const InsertArgs& a) { return a.ds.nch * 16 >= GT_LONG && a.alpha >= GT_ALPHA; }

hipError_t launch_forward_prune_gram(int dtype, const InsertArgs& a, hipStream_t st) {
    if (a.B <= 0) return hipSuccess;
    if (dtype == JX_U8) return launch_forward_gram_dt<JX_U8>(a, st);
    if (dtype == JX_F16) return launch_forward_gram_dt<JX_F16>(a, st);
    return two_parts_first(a) ? launch_forward_gram_dt<JX_F32, true>(a, st) : launch_forward_gram_dt<JX_F32>(a, st);
}

hipError_t launch_reverse_merge_gram(int dtype, const InsertArgs& a, hipStream_t st) {
    if (dtype == JX_U8) return launch_reverse_gram_dt<JX_U8>(a, st);
    if (dtype == JX_F16) return launch_reverse_gram_dt<JX_F16>(a, st);
    return two_parts_first(a) ? launch_reverse_gram_dt<JX_F32, true>(a, st) : launch_reverse_gram_dt<JX_F32>(a, st);
}

}  // namespace jx
