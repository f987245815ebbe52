// RaBitQ pipeline (Sec. 5.1): rotation GEMM on the matrix cores, encoder,
// integer query records, exact re-rank.
//
//   rotate      out = (in - c) P^T   queries and 1-bit codes: bfloat16 MFMA on three parts of
//               each float32 value, 128x128 tile per workgroup; codes of more
//               bits: float32 MFMA, 128x64.  K staged through LDS in slabs of
//               32; the centroid is subtracted while staging.
//   encode      one wavefront per vector: 1-bit codes via ballot, more bits with
//               the max-abs grid scale, or a workgroup with the max-cosine one;
//               data_add, data_rescale in double.
//   query prep  one wavefront per query: min/max, B_q-bit integer query,
//               nibble planes (4-bit codes) or bit planes (1-bit codes).
//   rerank      one wavefront per query: exact float32 squared L2 of the first
//               `rerank` frontier entries against the original query, sorted by
//               (distance, id).
#include "jx_distance.h"

namespace jx {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float rq_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 rq_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 rq_bf16x2 __attribute__((ext_vector_type(2)));

#define GT 128
#define GK 32
#define GLD 36               // floats of a staged row of the float32 form, padded
#define GPIECE 576            // 32 rows x 16 operand bytes, padded: 64 bytes further on in the banks from piece to piece
#define GBLOCK (12 * GPIECE)  // operand pieces of 32 rows and a slab: [step][part][half]

// Four float32 values as three bfloat16 parts each, whose sum they are exactly (8 bits of the significand in each; values below
// 2^-110 lose what lies below 2^-134)
__device__ __forceinline__ void rotate_stage(uint8_t* at, float v0, float v1, float v2, float v3) {
#pragma unroll
    for (int part = 0; part < 3; part++) {
        const rq_f32x2 x = {v0, v1}, y = {v2, v3};
        const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, rq_bf16x2));
        const uint32_t k = __builtin_bit_cast(uint32_t, __builtin_convertvector(y, rq_bf16x2));
        v0 -= __uint_as_float(h << 16);
        v1 -= __uint_as_float(h & 0xFFFF0000u);
        v2 -= __uint_as_float(k << 16);
        v3 -= __uint_as_float(k & 0xFFFF0000u);
        *reinterpret_cast<uint2*>(at + part * 2 * GPIECE) = make_uint2(h, k);
    }
}

template <int IN>
__device__ __forceinline__ float4 rotate_load(const void* in_v, const size_t at) {
    if (IN == JX_F16) {
        const _Float16* hp = reinterpret_cast<const _Float16*>(in_v) + at;
        return make_float4((float)hp[0], (float)hp[1], (float)hp[2], (float)hp[3]);
    } else if (IN == JX_U8) {
        const uint8_t* bp = reinterpret_cast<const uint8_t*>(in_v) + at;
        return make_float4((float)bp[0], (float)bp[1], (float)bp[2], (float)bp[3]);
    } else {
        return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(in_v) + at);
    }
}

// IN: storage type of the input rows (JX_F32, JX_F16, JX_U8); all three convert to float32 exactly.
// Six products of the parts (those of weight 2^-17 and above; what is left out is at most 2^-24 of a product) take 192 cycles
// for 16 coordinates where v_mfma_f32_32x32x2_f32 takes 512; every 32 coordinates have a sum of their own, so the result is
// nearer to 64 bits than that instruction's: error relative to the root mean square of a row, root mean square / largest,
// d = 128 8.1e-8 / 7.1e-7 (2.0e-7 / 2.3e-6 before), d = 960 1.3e-7 / 2.1e-6 (5.6e-7 / 9.4e-6).  Values of 3.39e38 and more
// round to an infinite part: elements that do not come out finite are summed again in plain float32.
// Bound: matrix instructions (1,536 cycles a slab and wavefront) and the vector instructions of the split (1,200), which
// overlap in part.  10,000 x 960 226 -> 149 us, 5,000 x 1536 235 -> 145, 50,000 x 960 717.
template <int IN>
__global__ void __launch_bounds__(256, 2) rotate_gemm_kernel(const void* __restrict__ in_v, long long n, int d,
                                                             const float* __restrict__ P, const float* __restrict__ c,
                                                             float* __restrict__ out) {
    __shared__ __align__(16) uint8_t As[4 * GBLOCK];
    __shared__ __align__(16) uint8_t Bs[4 * GBLOCK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const long long m0 = (long long)blockIdx.y * GT;
    const int n0 = blockIdx.x * GT;
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

    // a slab on its way in registers while the one before it is multiplied; rows beyond the last are read again, and what
    // comes of them is not stored.  d is a multiple of 32: every slab is whole
    const int srow = tid >> 3, piece = tid & 7, c4 = piece * 4;
    float4 pa[4], pb[4], pc;
    auto fetch = [&](const int k0) __attribute__((always_inline)) {
        pc = *reinterpret_cast<const float4*>(c + k0 + c4);
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const long long ra = m0 + srow + 32 * t < n ? m0 + srow + 32 * t : n - 1;
            const int rb = n0 + srow + 32 * t < d ? n0 + srow + 32 * t : d - 1;
            pa[t] = rotate_load<IN>(in_v, (size_t)ra * d + k0 + c4);
            pb[t] = *reinterpret_cast<const float4*>(P + (size_t)rb * d + k0 + c4);
        }
    };
    fetch(0);
    const int to = ((piece >> 2) * 6 + ((piece >> 1) & 1)) * GPIECE + (piece & 1) * 8 + srow * 16;
    const int from = (lane >> 5) * GPIECE + (lane & 31) * 16;
    for (int k0 = 0; k0 < d; k0 += GK) {
#pragma unroll
        for (int t = 0; t < 4; t++) {
            rotate_stage(As + t * GBLOCK + to, pa[t].x - pc.x, pa[t].y - pc.y, pa[t].z - pc.z, pa[t].w - pc.w);
            rotate_stage(Bs + t * GBLOCK + to, pb[t].x, pb[t].y, pb[t].z, pb[t].w);
        }
        __syncthreads();
        if (k0 + GK < d) fetch(k0 + GK);
#pragma unroll
        for (int mi = 0; mi < 2; mi++) {
            rq_bf16x8 a[2][3];
#pragma unroll
            for (int q = 0; q < 6; q++) a[q / 3][q % 3] = *reinterpret_cast<const rq_bf16x8*>(As + (wm * 2 + mi) * GBLOCK + from + q * 2 * GPIECE);
#pragma unroll
            for (int ni = 0; ni < 2; ni++) {
                f32x16 part;
#pragma unroll
                for (int e = 0; e < 16; e++) part[e] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 2; ks++) {
                    rq_bf16x8 b[3];
#pragma unroll
                    for (int q = 0; q < 3; q++) b[q] = *reinterpret_cast<const rq_bf16x8*>(Bs + (wn * 2 + ni) * GBLOCK + from + (ks * 3 + q) * 2 * GPIECE);
                    // the smallest products first
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][2], b[0], part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[2], part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][1], b[1], part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][1], b[0], part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[1], part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][0], b[0], part, 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < 16; e++) acc[mi][ni][e] += part[e];
            }
        }
        __syncthreads();
    }
    bool odd = false;
#pragma unroll
    for (int mi = 0; mi < 2; mi++)
#pragma unroll
        for (int ni = 0; ni < 2; ni++)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const long long row = m0 + wm * 64 + mi * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                const int col = n0 + wn * 64 + ni * 32 + (lane & 31);
                if (row < n && col < d) {
                    const float v = acc[mi][ni][e];
                    out[(size_t)row * d + col] = v;
                    odd = odd || !(fabsf(v) < __builtin_inff());
                }
            }
    if (!__syncthreads_or(odd)) return;
    __threadfence_block();
    for (int i = tid; i < GT * GT; i += 256) {
        const long long row = m0 + i / GT;
        const int col = n0 + i % GT;
        if (row >= n || col >= d || fabsf(out[(size_t)row * d + col]) < __builtin_inff()) continue;
        float s = 0.f;
        for (int k = 0; k < d; k += 4) {
            const float4 x = rotate_load<IN>(in_v, (size_t)row * d + k), p = *reinterpret_cast<const float4*>(P + (size_t)col * d + k);
            s = fmaf(x.x - c[k], p.x, s);
            s = fmaf(x.y - c[k + 1], p.y, s);
            s = fmaf(x.z - c[k + 2], p.z, s);
            s = fmaf(x.w - c[k + 3], p.w, s);
        }
        out[(size_t)row * d + col] = s;
    }
}

// The same by v_mfma_f32_32x32x2_f32, for codes of more than one bit.  Which grid point is nearest is often decided by the last
// bits of the rotated vector: between the two forms 6e-6 of the 4-bit codes of a set differ and 2.1e-5 of the 8-bit codes, and a
// vector whose best two grid scales are nearly equal gets another factor along with them.  So codes stay what they were for
// indices that are filled over time.  Tiles of 128 rows and TN columns, each wavefront 64 x TN / 2 of them.
// Bound: the float32 matrix instructions (512 cycles for 32 x 32 x 16).  A float4 of pb goes to LDS by its components: stored as a
// whole the array stays in scratch memory, every slab waits for it, and 8,000 x 1536 take 369 us (328 with 64 columns, 311
// with 128).
template <int IN, int TN>
__global__ void __launch_bounds__(256) rotate_f32_kernel(const void* __restrict__ in_v, long long n, int d,
                                                         const float* __restrict__ P, const float* __restrict__ c,
                                                         float* __restrict__ out) {
    __shared__ __align__(16) float As[GT][GLD];
    constexpr int NJ = TN / 64;  // tiles of 32 columns of a wavefront
    __shared__ __align__(16) float Bs[TN][GLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const long long m0 = (long long)blockIdx.y * GT;
    const int n0 = blockIdx.x * TN;
    f32x16 acc[2][NJ];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < NJ; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

    // a slab on its way in registers while the one before it is multiplied
    const int srow = tid >> 3, c4 = (tid & 7) * 4;
    float4 pa[4], pb[TN / 32], pc;
    auto fetch = [&](const int k0) __attribute__((always_inline)) {
        pc = *reinterpret_cast<const float4*>(c + k0 + c4);
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const long long ra = m0 + srow + 32 * t < n ? m0 + srow + 32 * t : n - 1;
            pa[t] = rotate_load<IN>(in_v, (size_t)ra * d + k0 + c4);
        }
#pragma unroll
        for (int t = 0; t < TN / 32; t++) {
            const int rb = n0 + srow + 32 * t < d ? n0 + srow + 32 * t : d - 1;
            pb[t] = *reinterpret_cast<const float4*>(P + (size_t)rb * d + k0 + c4);
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < d; k0 += GK) {
#pragma unroll
        for (int t = 0; t < 4; t++)
            *reinterpret_cast<float4*>(&As[srow + 32 * t][c4]) = make_float4(pa[t].x - pc.x, pa[t].y - pc.y, pa[t].z - pc.z, pa[t].w - pc.w);
#pragma unroll
        for (int t = 0; t < TN / 32; t++) *reinterpret_cast<float4*>(&Bs[srow + 32 * t][c4]) = make_float4(pb[t].x, pb[t].y, pb[t].z, pb[t].w);
        __syncthreads();
        if (k0 + GK < d) fetch(k0 + GK);
#pragma unroll
        for (int s8 = 0; s8 < GK / 8; s8++) {
            float4 af[2], bf[NJ];
#pragma unroll
            for (int s = 0; s < NJ; s++) bf[s] = *reinterpret_cast<const float4*>(&Bs[wn * (TN / 2) + s * 32 + (lane & 31)][8 * s8 + 4 * (lane >> 5)]);
#pragma unroll
            for (int s = 0; s < 2; s++) af[s] = *reinterpret_cast<const float4*>(&As[wm * 64 + s * 32 + (lane & 31)][8 * s8 + 4 * (lane >> 5)]);
#pragma unroll
            for (int mi = 0; mi < 2; mi++)
#pragma unroll
                for (int ni = 0; ni < NJ; ni++) {
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi].x, bf[ni].x, acc[mi][ni], 0, 0, 0);
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi].y, bf[ni].y, acc[mi][ni], 0, 0, 0);
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi].z, bf[ni].z, acc[mi][ni], 0, 0, 0);
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi].w, bf[ni].w, acc[mi][ni], 0, 0, 0);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int mi = 0; mi < 2; mi++)
#pragma unroll
        for (int ni = 0; ni < NJ; ni++)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const long long row = m0 + wm * 64 + mi * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                const int col = n0 + wn * (TN / 2) + ni * 32 + (lane & 31);
                if (row < n && col < d) out[(size_t)row * d + col] = acc[mi][ni][e];
            }
}

// Tiles of 64 columns or of 128: rounds of 256 workgroups, a round of wide tiles takes 1.9 times as long.  64 / 128 columns in us:
// 12,500 x 960 207 / 261 (6 rounds / 4), 50,000 x 960 763 / 812 (23 / 13), 5,000 x 1536 220 / 215 (4 / 2), 8,000 x 1536 328 / 311
// (6 / 3), 20,000 x 1536 790 / 797 (15 / 8), 50,000 x 1536 1,933 / 1,878 (37 / 19), 1,000 x 128 13 / 14 (1 / 1)
static bool rotate_narrow(long long n, int d) {
    const long long rows = (n + GT - 1) / GT;
    const long long narrow = (rows * ((d + 63) / 64) + 255) / 256, wide = (rows * ((d + 127) / 128) + 255) / 256;
    return narrow * 21 < wide * 40;
}

template <int TN>
static void launch_rotate_f32(const void* in, int in_dtype, long long n, int d, const float* P, const float* c, float* out, hipStream_t st) {
    const dim3 grid((unsigned)((d + TN - 1) / TN), (unsigned)((n + GT - 1) / GT));
    if (in_dtype == JX_F16)
        hipLaunchKernelGGL((rotate_f32_kernel<JX_F16, TN>), grid, dim3(256), 0, st, in, n, d, P, c, out);
    else if (in_dtype == JX_U8)
        hipLaunchKernelGGL((rotate_f32_kernel<JX_U8, TN>), grid, dim3(256), 0, st, in, n, d, P, c, out);
    else
        hipLaunchKernelGGL((rotate_f32_kernel<JX_F32, TN>), grid, dim3(256), 0, st, in, n, d, P, c, out);
}

hipError_t launch_rotate(const void* in, int in_dtype, long long n, int d, const float* P, const float* c, float* out, bool f32,
                         hipStream_t st) {
    if (n <= 0) return hipSuccess;
    dim3 grid((unsigned)((d + GT - 1) / GT), (unsigned)((n + GT - 1) / GT));
    if (f32) {
        if (rotate_narrow(n, d)) launch_rotate_f32<64>(in, in_dtype, n, d, P, c, out, st);
        else launch_rotate_f32<128>(in, in_dtype, n, d, P, c, out, st);
        return hipGetLastError();
    }
    if (in_dtype == JX_F16)
        hipLaunchKernelGGL(rotate_gemm_kernel<JX_F16>, grid, dim3(256), 0, st, in, n, d, P, c, out);
    else if (in_dtype == JX_U8)
        hipLaunchKernelGGL(rotate_gemm_kernel<JX_U8>, grid, dim3(256), 0, st, in, n, d, P, c, out);
    else
        hipLaunchKernelGGL(rotate_gemm_kernel<JX_F32>, grid, dim3(256), 0, st, in, n, d, P, c, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ encoder

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += shfl_xor(v, m);
    return v;
}
__device__ __forceinline__ float wave_max_f32(float v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v = fmaxf(v, shfl_xor(v, m));
    return v;
}
__device__ __forceinline__ float wave_min_f32(float v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v = fminf(v, shfl_xor(v, m));
    return v;
}

// Code layout: 1-bit: coordinate i is bit i%32 of dword i/32.  4-bit: coordinate i
// is nibble i%8 of dword i/8 (so even coordinates sit in low nibbles of a byte).
__global__ void __launch_bounds__(256) encode_kernel(EncodeArgs a) {
    const long long v = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= a.n) return;
    const int lane = lane_id();
    const float* r = a.rot + (size_t)v * a.d;
    uint8_t* code = a.codes + (size_t)v * a.code_stride;
    double l2 = 0.0, ip = 0.0;
    if (a.bits == 1) {
        for (int c0 = 0; c0 < a.d; c0 += 64) {
            const int i = c0 + lane;
            const float x = i < a.d ? r[i] : -1.0f;
            const bool pos = i < a.d && x >= 0.0f;
            const uint64_t m = ballot(pos);
            if (i < a.d) {
                l2 += (double)x * (double)x;
                ip += 0.5 * fabs((double)x);
            }
            if (lane == 0) *reinterpret_cast<uint32_t*>(code + c0 / 8) = (uint32_t)m;
            if (lane == 1 && c0 + 32 < a.d) *reinterpret_cast<uint32_t*>(code + c0 / 8 + 4) = (uint32_t)(m >> 32);
        }
    } else {
        const int half = 1 << (a.bits - 1);
        float amax = 0.f;
        for (int i = lane; i < a.d; i += 64) amax = fmaxf(amax, fabsf(r[i]));
        amax = wave_max_f32(amax);
        const float t = amax > 0.f ? __fdiv_rn((float)half - 0.5f, amax) : 0.f;
        const double cb = ((double)(1 << a.bits) - 1.0) * 0.5;
        // 32 / bits consecutive coordinates per lane -> one dword (field i % per of dword i / per)
        const int per = 32 / a.bits;
        for (int c0 = 0; c0 < a.d; c0 += 64 * per) {
            const int i0 = c0 + lane * per;
            if (i0 < a.d) {
                uint32_t w = 0;
                for (int j = 0; j < per; j++) {
                    const float x = r[i0 + j];
                    float lvf = floorf(__fmul_rn(t, fabsf(x)));
                    int lv = (int)lvf;
                    lv = lv > half - 1 ? half - 1 : (lv < 0 ? 0 : lv);
                    const int u = x >= 0.0f ? half + lv : half - 1 - lv;
                    w |= (uint32_t)u << (a.bits * j);
                    l2 += (double)x * (double)x;
                    ip += ((double)u - cb) * (double)x;
                }
                *reinterpret_cast<uint32_t*>(code + (size_t)i0 * a.bits / 8) = w;
            }
        }
    }
    l2 = wave_sum_f64(l2);
    ip = wave_sum_f64(ip);
    for (int b = a.code_bytes + lane * 4; b < a.pad_to; b += 256) *reinterpret_cast<uint32_t*>(code + b) = 0u;
    if (lane == 0) {
        float* m = reinterpret_cast<float*>(a.meta + (size_t)v * a.meta_stride);
        m[0] = l2 > 0.0 ? (float)l2 : 0.f;
        m[1] = l2 > 0.0 ? (float)(-2.0 * l2 / ip) : 0.f;
        for (int b = 0; b < a.meta_pad; b += 4) m[2 + b / 4] = 0.f;
    }
}

// ---- max-cosine rule (m > 1): the grid point whose direction is closest to r.
// One workgroup per vector.  The grid scale t steps coordinate i to level j at the breakpoint t = j/|r_i|
// (j = 1 .. 2^(m-1)-1); after the breakpoints <= t have been applied,
//     <xbar,|r|> = l1/2 + sum_j PrefA[cnt_j(t)],   ||xbar||^2 = d/4 + sum_j 2j cnt_j(t),
// where cnt_j(t) counts the level-j breakpoints <= t and PrefA are prefix sums of the magnitudes in descending
// order.  So only the d magnitudes are sorted (bitonic network in LDS); the level-j breakpoints j/|r|_(p) are then
// already ascending in p.  Breakpoints are compared as products, j |r|_(p') against j' |r|_(p), which are exact in double
// (two different quotients of integers below 8 and float32 numbers differ by 2^-27 of their size, so the rounded quotients
// compare alike).  A thread takes consecutive breakpoints of one level and moves its counts along: the state at the end of
// each group of equal t.  The largest cosine wins, the smallest t among equals, and t -> 0+ competes.  The level of a
// coordinate is then the number of its own breakpoints that are <= t.
//
// Few breakpoints can win.  The state is taken at 256 values t_g (64 for few dimensions) first, a binary search per level and
// thread.  A breakpoint in (t_g, t_g+1] of level j has |r| < j / t_g, so where such breakpoints add x to ||xbar||^2 they add
// less than x / (2 t_g) to <xbar,|r|>, and (ip_g + x / (2 t_g)) / sqrt(nn_g + x) falls and then rises with x: the larger of its
// values at both ends bounds every cosine of the interval.  Both ends are close to cosines that are reached, an interval a
// hundredth of t wide is bounded to some 1e-4, and what is left around the maximum (some 600 of 6,720 breakpoints at d =
// 960) is evaluated exactly, all threads at once.  (A bound by the sums at both ends alone leaves most breakpoints in.)
// Bound: vector instructions of the searches and of the sort.  50,000 vectors of d = 960, 4 bits 6,960 -> 1,010 us; before
// that every breakpoint was evaluated, a thread moving its counts along consecutive ones of a level.  Whole quantisation,
// rotation included: 53,353 x 96 1,086 -> 561, 50,000 x 128 1,180 -> 546, 30,000 x 256 1,260 -> 429, 20,000 x 512 1,620 -> 406,
// 2 bits 50,000 x 1536 4,622 -> 3,652
#define MC_CAP 8192   // breakpoints per vector
#define MC_DMAX 4096  // dimensions

__device__ __forceinline__ double block_scan_incl(double v, double* ws, int tid) {
    // inclusive scan over the 256 threads of the workgroup
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        double o = __shfl_up(v, s, 64);
        if (lane >= s) v += o;
    }
    if (lane == 63) ws[wave] = v;
    __syncthreads();
    double off = 0.0;
    for (int w = 0; w < wave; w++) off += ws[w];
    __syncthreads();
    return v + off;
}

// one stage of the network below: entry i = tid V + r against entry i ^ J, descending where i & K is 0
template <int V, int K, int J>
__device__ __forceinline__ void sort_stage(float (&v)[V], float* sa, const int tid) {
    if constexpr (J < V) {
#pragma unroll
        for (int r = 0; r < V; r++)
            if ((r & J) == 0) {
                const bool down = K < V ? (r & K) == 0 : (tid & (K / V)) == 0;
                const float hi = fmaxf(v[r], v[r | J]), lo = fminf(v[r], v[r | J]);
                v[r] = down ? hi : lo;
                v[r | J] = down ? lo : hi;
            }
    } else {
        const bool top = ((tid & (J / V)) == 0) == ((tid & (K / V)) == 0);
        float o[V];
        if constexpr (J / V < 64) {
#pragma unroll
            for (int r = 0; r < V; r++) o[r] = __uint_as_float(lane_xor_u32<J / V>(__float_as_uint(v[r])));
        } else {  // another wavefront's
#pragma unroll
            for (int r = 0; r < V; r++) sa[r * 256 + tid] = v[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < V; r++) o[r] = sa[r * 256 + (tid ^ (J / V))];
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < V; r++) v[r] = top ? fmaxf(v[r], o[r]) : fminf(v[r], o[r]);
    }
    if constexpr (J > 1)
        sort_stage<V, K, J / 2>(v, sa, tid);
    else if constexpr (K < V * 256)
        sort_stage<V, K * 2, K>(v, sa, tid);
}

// NL = 2^(bits-1) - 1 levels, V magnitudes per thread (256 V >= d)
template <int NL, int V>
__global__ void __launch_bounds__(256) encode_maxcos_kernel(EncodeArgs a) {
    constexpr int half = NL + 1, dpad = 256 * V;
    __shared__ __align__(16) float sa[dpad];  // magnitudes, descending
    __shared__ double pref[dpad + 1];         // prefix sums of sa
    __shared__ double ws[8];
    __shared__ double st_ip[256], st_nn[256];  // state at t_g
    __shared__ uint16_t st_cnt[256 * NL];
    __shared__ uint64_t keep[4];
    __shared__ double red_c[4], red_t[4];
    __shared__ float red_a[4];
    __shared__ int red_j[4];
    __shared__ int s_npos;
    __shared__ double s_l1, s_l2, s_ip;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long v = blockIdx.x;
    const float* r = a.rot + (size_t)v * a.d;
    uint8_t* code = a.codes + (size_t)v * a.code_stride;

    // ---- sums, magnitudes
    double l1 = 0.0, l2 = 0.0;
    int npos_t = 0;
    float mag[V];
#pragma unroll
    for (int q = 0; q < V; q++) {
        const int i = tid + 256 * q;
        mag[q] = i < a.d ? fabsf(r[i]) : 0.f;
        const double x = (double)mag[q];
        l1 += x;
        l2 += x * x;
        npos_t += mag[q] > 0.f ? 1 : 0;
    }
    {   // block sums (fixed order)
        const double t1 = block_scan_incl(l1, ws, tid);
        if (tid == 255) s_l1 = t1;
        const double t2 = block_scan_incl(l2, ws, tid);
        if (tid == 255) s_l2 = t2;
        const double t3 = block_scan_incl((double)npos_t, ws, tid);
        if (tid == 255) s_npos = (int)t3;
    }
    // ---- bitonic sort, descending: in registers, through LDS only between wavefronts
    sort_stage<V, 2, 1>(mag, sa, tid);
#pragma unroll
    for (int q = 0; q < V; q++) sa[tid * V + q] = mag[q];
    // ---- prefix sums (thread t owns V consecutive entries)
    {
        double loc = 0.0;
#pragma unroll
        for (int q = 0; q < V; q++) loc += (double)mag[q];
        double run = block_scan_incl(loc, ws, tid) - loc;
        if (tid == 0) pref[0] = 0.0;
#pragma unroll
        for (int q = 0; q < V; q++) {
            run += (double)mag[q];
            pref[tid * V + q + 1] = run;
        }
    }
    __syncthreads();
    const int npos = s_npos;  // the zeros sit behind the npos positive magnitudes
    const double ip0 = 0.5 * s_l1, nn0 = 0.25 * (double)a.d;
    // ---- states at t_0 = 0, a geometric grid from just below the first breakpoint to 8 / (the median magnitude), and infinity
    const int G = V == 1 ? 64 : 256;
    double t_g = 0.0, ip_g = ip0, nn_g = nn0, c_g = -1.0;
    if (tid < G) {
        const float first = 0.99f / sa[0], last = 8.f / sa[npos >> 1 > 0 ? (npos >> 1) - 1 : 0];
        const float grow = log2f(last / first) / (float)(G - 3);
        float t = tid == 0 ? 0.f : first * exp2f(grow * (float)(tid - 1));
        if (tid == G - 1 || !(t < __builtin_inff())) t = __builtin_inff();
        t_g = (double)t;
        int cnt[NL];
#pragma unroll
        for (int jj = 0; jj < NL; jj++) cnt[jj] = 0;
        if (t == __builtin_inff()) {
#pragma unroll
            for (int jj = 0; jj < NL; jj++) cnt[jj] = npos;
        } else {
            // all levels side by side, a chain of LDS reads for one; behind npos stand zeros, which reach no level
            for (int step = dpad >> 1, end = 0; !end; step = step > 1 ? step >> 1 : 0) {
                end = step == 0;  // dpad entries have dpad + 1 places: one more step of one
                const int by = end ? 1 : step;
#pragma unroll
                for (int jj = 0; jj < NL; jj++)
                    if ((double)(jj + 1) <= t_g * (double)sa[cnt[jj] + by - 1]) cnt[jj] += by;
            }
        }
#pragma unroll
        for (int jj = 0; jj < NL; jj++) {
            st_cnt[jj * 256 + tid] = (uint16_t)cnt[jj];
            ip_g += pref[cnt[jj]];
            nn_g += 2.0 * (double)(jj + 1) * (double)cnt[jj];
        }
        st_ip[tid] = ip_g;
        st_nn[tid] = nn_g;
        c_g = ip_g / sqrt(nn_g);
    }
    {
        double most = c_g;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const double o = shfl_xor(most, m);
            most = o > most ? o : most;
        }
        if (lane == 0) ws[wave] = most;
    }
    __syncthreads();
    {   // intervals that may hold the largest cosine; comparisons with NaN keep them
        double least = ws[0];
        for (int w = 1; w < 4; w++) least = ws[w] > least ? ws[w] : least;
        least *= 1.0 - 1e-9;
        bool on = false;
        if (tid < G - 1) {
            const double next = st_nn[tid + 1], x = next - nn_g;
            const double end = (ip_g + 0.5 * x / t_g) / sqrt(next);  // t_0: infinite
            on = x != 0.0 && !(c_g < least && end < least);
        }
        const uint64_t m = ballot(on);
        if (lane == 0) keep[wave] = m;
    }
    __syncthreads();
    int g0 = 256, g1 = -1;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        const uint64_t m = keep[w];
        if (m) {
            if (g0 == 256) g0 = w * 64 + __builtin_ctzll(m);
            g1 = w * 64 + 63 - __builtin_clzll(m);
        }
    }
    // ---- the breakpoints in (t_g0, t_g1 + 1]: of every level consecutive ones
    int lo[NL], hi[NL], total = 0, widest = 0;
#pragma unroll
    for (int jj = 0; jj < NL; jj++) {
        lo[jj] = g1 < 0 ? 0 : (int)st_cnt[jj * 256 + g0];
        hi[jj] = g1 < 0 ? 0 : (int)st_cnt[jj * 256 + g1 + 1];
        if (hi[jj] < lo[jj]) hi[jj] = lo[jj];  // rows with NaN
        total += hi[jj] - lo[jj];
        widest = hi[jj] - lo[jj] > widest ? hi[jj] - lo[jj] : widest;
    }
    int top = 1;
    while (2 * top <= widest) top *= 2;
    double best = -1.0, best_t = __builtin_inf();
    float best_a = 1.f;
    int best_j = 0;
    for (int k = tid; k < total; k += 256) {
        int lev = 0, p = k;
#pragma unroll
        for (int jj = 0; jj < NL; jj++)
            if (lev == jj) {
                const int n = hi[jj] - lo[jj];
                if (p < n) p += lo[jj];
                else {
                    p -= n;
                    lev = jj + 1;
                    continue;
                }
                break;
            }
        const float Af = sa[p];
        const double A = (double)Af, J = (double)(lev + 1);
        // counts at the end of the group of equal t, inside the window
        int cnt[NL];
#pragma unroll
        for (int jj = 0; jj < NL; jj++) cnt[jj] = lo[jj];
        for (int step = top; step >= 1; step >>= 1)
#pragma unroll
            for (int jj = 0; jj < NL; jj++)
                if (cnt[jj] + step <= hi[jj] && (double)(jj + 1) * A <= J * (double)sa[cnt[jj] + step - 1]) cnt[jj] += step;
        double ip = ip0, nn = nn0;
#pragma unroll
        for (int jj = 0; jj < NL; jj++) {
            ip += pref[cnt[jj]];
            nn += 2.0 * (double)(jj + 1) * (double)cnt[jj];
        }
        const double c = ip / sqrt(nn);
        if (c >= best) {
            const double t = J / A;
            if (c > best || t < best_t) {
                best = c;
                best_t = t;
                best_a = Af;
                best_j = lev + 1;
            }
        }
    }
    // largest cosine, the smallest t among equals
    auto better = [&](const double oc, const double ot, const float oa, const int oj) {
        if (oc > best || (oc == best && ot < best_t)) {
            best = oc;
            best_t = ot;
            best_a = oa;
            best_j = oj;
        }
    };
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const double oc = shfl_xor(best, m), ot = shfl_xor(best_t, m);
        const float oa = shfl_xor(best_a, m);
        const int oj = shfl_xor(best_j, m);
        better(oc, ot, oa, oj);
    }
    if (lane == 0) {
        red_c[wave] = best;
        red_t[wave] = best_t;
        red_a[wave] = best_a;
        red_j[wave] = best_j;
    }
    __syncthreads();
    best = -1.0;
    best_t = __builtin_inf();
    best_a = 1.f;
    best_j = 0;
    for (int w = 0; w < 4; w++) better(red_c[w], red_t[w], red_a[w], red_j[w]);
    // the all-zero-level grid (t -> 0+) competes too; a later cosine must be strictly larger
    if (!(npos > 0 && best > ip0 / sqrt(nn0))) best_j = 0;
    // level lv + 1 is reached where (lv + 1) / |r_i| <= j / a
    const double bj = (double)best_j, ba = (double)best_a;
    // ---- codes: 32 / bits consecutive coordinates per thread -> one dword
    const double cb = ((double)(1 << a.bits) - 1.0) * 0.5;
    const int per = 32 / a.bits;
    double ip = 0.0;
    for (int i0 = tid * per; i0 < a.d; i0 += 256 * per) {
        uint32_t w = 0;
        for (int j = 0; j < per; j++) {
            const float x = r[i0 + j];
            const double ax = fabs((double)x);
            int lv = 0;
            if (ax > 0.0)
                while (lv + 1 < half && (double)(lv + 1) * ba <= bj * ax) lv++;
            const int u = x >= 0.0f ? half + lv : half - 1 - lv;
            w |= (uint32_t)u << (a.bits * j);
            ip += ((double)u - cb) * (double)x;
        }
        *reinterpret_cast<uint32_t*>(code + (size_t)i0 * a.bits / 8) = w;
    }
    const double tip = block_scan_incl(ip, ws, tid);
    if (tid == 255) s_ip = tip;
    __syncthreads();
    for (int b = a.code_bytes + tid * 4; b < a.pad_to; b += 1024) *reinterpret_cast<uint32_t*>(code + b) = 0u;
    if (tid == 0) {
        float* m = reinterpret_cast<float*>(a.meta + (size_t)v * a.meta_stride);
        m[0] = s_l2 > 0.0 ? (float)s_l2 : 0.f;
        m[1] = s_l2 > 0.0 ? (float)(-2.0 * s_l2 / s_ip) : 0.f;
        for (int b = 0; b < a.meta_pad; b += 4) m[2 + b / 4] = 0.f;
    }
}

hipError_t launch_encode(const EncodeArgs& a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    if (a.bits > 1 && a.rule == JX_RULE_MAXCOS) {
        const int nl = (1 << (a.bits - 1)) - 1;
        if ((a.bits != 4 && a.bits != 2) || a.d * nl > MC_CAP || a.d > MC_DMAX) return hipErrorInvalidValue;
        const dim3 grid((unsigned)a.n), block(256);
        if (a.bits == 4) {  // at most 1,170 dimensions
            if (a.d <= 256) hipLaunchKernelGGL((encode_maxcos_kernel<7, 1>), grid, block, 0, st, a);
            else if (a.d <= 512) hipLaunchKernelGGL((encode_maxcos_kernel<7, 2>), grid, block, 0, st, a);
            else if (a.d <= 1024) hipLaunchKernelGGL((encode_maxcos_kernel<7, 4>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((encode_maxcos_kernel<7, 8>), grid, block, 0, st, a);
        } else {
            if (a.d <= 256) hipLaunchKernelGGL((encode_maxcos_kernel<1, 1>), grid, block, 0, st, a);
            else if (a.d <= 512) hipLaunchKernelGGL((encode_maxcos_kernel<1, 2>), grid, block, 0, st, a);
            else if (a.d <= 1024) hipLaunchKernelGGL((encode_maxcos_kernel<1, 4>), grid, block, 0, st, a);
            else if (a.d <= 2048) hipLaunchKernelGGL((encode_maxcos_kernel<1, 8>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((encode_maxcos_kernel<1, 16>), grid, block, 0, st, a);
        }
        return hipGetLastError();
    }
    hipLaunchKernelGGL(encode_kernel, dim3((unsigned)((a.n + 3) / 4)), dim3(256), 0, st, a);
    return hipGetLastError();
}

// 2-bit and 8-bit codes are searched as two planes of the 1-bit / 4-bit provider: u = lo + 2^f hi with f = 1 / 4.
// Natural packing (field i % per of dword i / per) <-> planes ([lo plane][hi plane], each plane_bytes long, a plane
// packed as 1-bit / 4-bit codes are).  Two natural dwords make one dword of each plane.
__device__ __forceinline__ uint32_t even_bits(uint32_t x) {  // bits 0,2,4,.. -> bits 0..15
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    x = (x | (x >> 8)) & 0x0000FFFFu;
    return x;
}
__device__ __forceinline__ uint32_t spread_bits(uint32_t x) {  // bits 0..15 -> bits 0,2,4,..
    x &= 0x0000FFFFu;
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    x = (x | (x << 1)) & 0x55555555u;
    return x;
}
__device__ __forceinline__ uint32_t low_nibbles(uint32_t x) {  // low nibble of each byte -> bits 0..15
    x &= 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    x = (x | (x >> 8)) & 0x0000FFFFu;
    return x;
}
__device__ __forceinline__ uint32_t spread_nibbles(uint32_t x) {  // nibbles 0..3 -> low nibble of bytes 0..3
    x &= 0x0000FFFFu;
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    return x;
}
__device__ __forceinline__ void split_pair(int bits, uint32_t n0, uint32_t n1, uint32_t* lo, uint32_t* hi) {
    if (bits == 2) {
        *lo = even_bits(n0) | (even_bits(n1) << 16);
        *hi = even_bits(n0 >> 1) | (even_bits(n1 >> 1) << 16);
    } else {
        *lo = low_nibbles(n0) | (low_nibbles(n1) << 16);
        *hi = low_nibbles(n0 >> 4) | (low_nibbles(n1 >> 4) << 16);
    }
}
__device__ __forceinline__ void join_pair(int bits, uint32_t lo, uint32_t hi, uint32_t* n0, uint32_t* n1) {
    if (bits == 2) {
        *n0 = spread_bits(lo) | (spread_bits(hi) << 1);
        *n1 = spread_bits(lo >> 16) | (spread_bits(hi >> 16) << 1);
    } else {
        *n0 = spread_nibbles(lo) | (spread_nibbles(hi) << 4);
        *n1 = spread_nibbles(lo >> 16) | (spread_nibbles(hi >> 16) << 4);
    }
}

// in place: natural codes at the start of each record -> two planes; one wavefront per record, staged in LDS
__global__ void __launch_bounds__(256) planarize_kernel(uint8_t* recs, long long n, int code_stride, int code_bytes, int plane_bytes,
                                                       int bits) {
    extern __shared__ __align__(16) uint32_t stage[];  // 4 x code_bytes / 4
    const long long v = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= n) return;
    const int lane = lane_id();
    uint32_t* mine = stage + (size_t)(threadIdx.x >> 6) * (code_bytes / 4);
    uint32_t* rec = reinterpret_cast<uint32_t*>(recs + (size_t)v * code_stride);
    const int nd = code_bytes / 4;  // natural dwords (even: dim % 32 == 0)
    for (int k = lane; k < nd; k += 64) mine[k] = rec[k];
    wave_sync();
    for (int k = lane; k < plane_bytes / 4; k += 64) {  // dword k of each plane, zero beyond the codes
        uint32_t lo = 0, hi = 0;
        if (2 * k + 1 < nd) split_pair(bits, mine[2 * k], mine[2 * k + 1], &lo, &hi);
        rec[k] = lo;
        rec[plane_bytes / 4 + k] = hi;
    }
}

hipError_t launch_planarize(uint8_t* recs, long long n, int code_stride, int code_bytes, int plane_bytes, int bits, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(planarize_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), (size_t)4 * code_bytes, st, recs, n, code_stride,
                       code_bytes, plane_bytes, bits);
    return hipGetLastError();
}

// records -> unpadded codes + meta
__global__ void __launch_bounds__(256) unpack_records_kernel(const uint8_t* recs, long long n, int code_stride, int code_bytes,
                                                            int meta_off, uint8_t* codes, float* meta, int planar_bits,
                                                            int plane_bytes) {
    const long long v = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= n) return;
    const int lane = lane_id();
    const uint8_t* rec = recs + (size_t)v * code_stride;
    if (planar_bits) {  // two planes -> natural packing
        const uint32_t* pl = reinterpret_cast<const uint32_t*>(rec);
        uint32_t* out = reinterpret_cast<uint32_t*>(codes + (size_t)v * code_bytes);
        for (int k = lane; 2 * k + 1 < code_bytes / 4; k += 64) {
            uint32_t n0, n1;
            join_pair(planar_bits, pl[k], pl[plane_bytes / 4 + k], &n0, &n1);
            out[2 * k] = n0;
            out[2 * k + 1] = n1;
        }
    } else
    for (int b = lane * 4; b < code_bytes; b += 256)
        *reinterpret_cast<uint32_t*>(codes + (size_t)v * code_bytes + b) = *reinterpret_cast<const uint32_t*>(rec + b);
    if (lane < 2) meta[2 * v + lane] = reinterpret_cast<const float*>(rec + meta_off)[lane];
}

hipError_t launch_unpack_records(const uint8_t* recs, long long n, int code_stride, int code_bytes, int meta_off,
                                 uint8_t* codes, float* meta, int planar_bits, int plane_bytes, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(unpack_records_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, recs, n, code_stride, code_bytes,
                       meta_off, codes, meta, planar_bits, plane_bytes);
    return hipGetLastError();
}

// unpadded codes + meta -> records (padding zeroed)
__global__ void __launch_bounds__(256) pack_records_kernel(uint8_t* recs, long long n, int code_stride, int code_bytes,
                                                          int meta_off, const uint8_t* codes, const float* meta) {
    const long long v = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= n) return;
    const int lane = lane_id();
    uint8_t* rec = recs + (size_t)v * code_stride;
    for (int b = lane * 4; b < code_stride; b += 256) {
        uint32_t w = 0;
        if (b < code_bytes) w = *reinterpret_cast<const uint32_t*>(codes + (size_t)v * code_bytes + b);
        else if (b == meta_off) w = __float_as_uint(meta[2 * v]);
        else if (b == meta_off + 4) w = __float_as_uint(meta[2 * v + 1]);
        *reinterpret_cast<uint32_t*>(rec + b) = w;
    }
}

hipError_t launch_pack_records(uint8_t* recs, long long n, int code_stride, int code_bytes, int meta_off,
                               const uint8_t* codes, const float* meta, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pack_records_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, recs, n, code_stride, code_bytes,
                       meta_off, codes, meta);
    return hipGetLastError();
}

// Sum of the code units of every record (codes in their natural packing: fields of `bits` bits), stored as a
// uint32 behind the two floats of the meta chunk: the estimator's sum(u) term then costs the search kernel nothing.
__global__ void __launch_bounds__(256) code_sums_kernel(uint8_t* recs, long long n, int code_stride, int code_bytes,
                                                       int meta_off, int bits) {
    const long long v = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= n) return;
    const int lane = lane_id();
    uint8_t* rec = recs + (size_t)v * code_stride;
    uint32_t s = 0;
    for (int b = lane * 4; b < code_bytes; b += 256) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(rec + b);
        if (bits == 1)
            s += (uint32_t)__builtin_popcount(w);
        else if (bits == 2)
            s += (uint32_t)__builtin_popcount(w & 0x55555555u) + 2u * (uint32_t)__builtin_popcount(w & 0xAAAAAAAAu);
        else if (bits == 4)
            s += __builtin_amdgcn_udot8(w, 0x11111111u, 0u, false);
        else
            s += __builtin_amdgcn_udot4(w, 0x01010101u, 0u, false);
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s += shfl_xor(s, m);
    if (lane == 0) *reinterpret_cast<uint32_t*>(rec + meta_off + 8) = s;
}

hipError_t launch_code_sums(uint8_t* recs, long long n, int code_stride, int code_bytes, int meta_off, int bits, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(code_sums_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, recs, n, code_stride, code_bytes,
                       meta_off, bits);
    return hipGetLastError();
}

// ------------------------------------------------------------------ query records

__global__ void __launch_bounds__(256) query_prep_kernel(QueryPrepArgs a) {
    const long long qi = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (qi >= a.nq) return;
    const int lane = lane_id();
    const float* q = a.rot + (size_t)qi * a.d;
    uint8_t* rec = a.qrecs + (size_t)qi * a.qrec_stride;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    double s = 0.0, s2 = 0.0;
    for (int i = lane; i < a.d; i += 64) {
        const float x = q[i];
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
        s += (double)x;
        s2 += (double)x * (double)x;
    }
    lo = wave_min_f32(lo);
    hi = wave_max_f32(hi);
    s = wave_sum_f64(s);
    s2 = wave_sum_f64(s2);
    const float levels = (float)((1 << a.qbits) - 1);
    const float delta = __fdiv_rn(__fsub_rn(hi, lo), levels);
    const double cb = ((double)(1 << a.bits) - 1.0) * 0.5;
    if (lane == 0) {
        float* hdr = reinterpret_cast<float*>(rec);
        hdr[0] = lo;
        hdr[1] = delta;
        hdr[2] = (float)s2;
        hdr[3] = (float)(cb * s);
    }
    const bool nib = a.bits >= 4;  // 4- and 8-bit codes: nibble planes; 1- and 2-bit codes: bit planes
    const int nplanes = nib ? 2 : a.qbits;
    // zero the padding of each plane (planes are whole 16-byte chunks)
    const int written = nib ? a.d / 2 : a.d / 8;
    for (int p = 0; p < nplanes; p++)
        for (int b = written + lane * 4; b < a.plane_stride; b += 256)
            *reinterpret_cast<uint32_t*>(rec + 16 + (size_t)p * a.plane_stride + b) = 0u;
    auto quant = [&](float x) -> uint32_t {
        if (!(delta > 0.f)) return 0u;
        float t = __fdiv_rn(__fsub_rn(x, lo), delta);
        t = floorf(__fadd_rn(t, 0.5f));
        t = t < 0.f ? 0.f : (t > levels ? levels : t);
        return (uint32_t)t;
    };
    if (nib) {
        // nibble planes: dword k holds coordinates 8k..8k+7; plane 0 = high nibbles, plane 1 = low nibbles
        for (int c0 = 0; c0 < a.d; c0 += 512) {
            const int i0 = c0 + lane * 8;
            if (i0 < a.d) {
                uint32_t wh = 0, wl = 0;
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    const uint32_t v = quant(q[i0 + j]);
                    wh |= (v >> 4) << (4 * j);
                    wl |= (v & 15u) << (4 * j);
                }
                *reinterpret_cast<uint32_t*>(rec + 16 + i0 / 2) = wh;
                *reinterpret_cast<uint32_t*>(rec + 16 + a.plane_stride + i0 / 2) = wl;
            }
        }
    } else {
        // bit planes: plane b, dword k, bit j = bit b of q_int[32k + j]
        for (int c0 = 0; c0 < a.d; c0 += 64) {
            const int i = c0 + lane;
            const uint32_t v = i < a.d ? quant(q[i]) : 0u;
            for (int b = 0; b < a.qbits; b++) {
                const uint64_t m = ballot(((v >> b) & 1u) != 0u);
                if (lane == 0) *reinterpret_cast<uint32_t*>(rec + 16 + (size_t)b * a.plane_stride + c0 / 8) = (uint32_t)m;
                if (lane == 1 && c0 + 32 < a.d)
                    *reinterpret_cast<uint32_t*>(rec + 16 + (size_t)b * a.plane_stride + c0 / 8 + 4) = (uint32_t)(m >> 32);
            }
        }
    }
}

hipError_t launch_query_prep(const QueryPrepArgs& a, hipStream_t st) {
    if (a.nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(query_prep_kernel, dim3((unsigned)((a.nq + 3) / 4)), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------ exact re-rank

struct RerankLds {
    uint64_t key[JX_MAX_L];
    uint64_t cand_key[64];
    uint32_t cand_id[64];
};

template <int KIND, int T, int CPL>
__global__ void __launch_bounds__(256) rerank_kernel(RerankArgs a) {
    __shared__ RerankLds lds[4];
    constexpr int G = 64 / T;
    constexpr int U0 = (8 / CPL) > 0 ? (8 / CPL) : 1;
    constexpr int U = U0 < (64 / G) ? U0 : (64 / G);
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int g = lane / T, lig = lane % T;
    const long long qi = (long long)blockIdx.x * 4 + wave;
    if (qi >= a.nq) return;
    RerankLds* L = &lds[wave];
    QueryRegs<KIND, CPL, 0> q;
    load_query<KIND, T, CPL, 0>(q, a.ds, qi, lig);
    const uint32_t* cand = a.cand + (size_t)qi * a.cand_stride;
    int m = 0;
    for (int c0 = 0; c0 < a.rr; c0 += 64) {
        const int j = c0 + lane;
        const uint32_t id = j < a.rr ? cand[j] : JX_NONE_ID;
        const uint64_t vm = ballot(id != JX_NONE_ID);
        const int nn = __builtin_popcountll(vm);
        if (nn == 0) break;  // the frontier is filled from the left
        if (id != JX_NONE_ID) L->cand_id[prefix_count(vm)] = id;
        wave_sync();
        for (int s0 = 0; s0 < nn; s0 += G * U) eval_batch<KIND, T, CPL, 0, U>(q, a.ds, s0, nn, L->cand_id, L->cand_key, g, lig);
        wave_sync();
        if (lane < nn) L->key[m + lane] = L->cand_key[lane] | 1ull;
        m += nn;
        wave_sync();
    }
    // rank sort by (distance, id); write the first k, pad what is left
    for (int j = m + lane; j < a.k; j += 64) {
        a.out_ids[qi * a.k + j] = JX_NONE_ID;
        a.out_dist[qi * a.k + j] = __builtin_inff();
    }
    for (int j = lane; j < m; j += 64) {
        const uint64_t kj = L->key[j];
        int rank = 0;
        for (int t = 0; t < m; t++) rank += (L->key[t] < kj) ? 1 : 0;
        if (rank < a.k) {
            a.out_ids[qi * a.k + rank] = key_id(kj);
            const uint32_t dc = key_dist(kj);
            a.out_dist[qi * a.k + rank] = (KIND == K_U8) ? (float)dc : ordered_to_f32(dc);
        }
    }
    if (a.stats && lane == 0) atomicAdd(&a.stats[(size_t)(qi & 63) * 16 + 2], (unsigned long long)m);
}

template <int KIND>
static hipError_t launch_rerank_shape(const RerankArgs& a, hipStream_t st) {
    dim3 grid((unsigned)((a.nq + 3) / 4)), block(256);
    const int nch = a.ds.nch;
#define JX_RR(T, C)                                                             \
    {                                                                           \
        hipLaunchKernelGGL((rerank_kernel<KIND, T, C>), grid, block, 0, st, a); \
        return hipGetLastError();                                               \
    }
    if (nch <= 8) JX_RR(4, 2)
    if (nch <= 16) JX_RR(8, 2)
    if (nch <= 32) JX_RR(16, 2)
    if (nch <= 64) JX_RR(32, 2)
    if (nch <= 128) JX_RR(64, 2)
    if (nch <= 256) JX_RR(64, 4)
    if (nch <= 384) JX_RR(64, 6)
#undef JX_RR
    return hipErrorInvalidValue;
}

hipError_t launch_rerank(int dtype, const RerankArgs& a, hipStream_t st) {
    if (a.nq <= 0) return hipSuccess;
    if (dtype == JX_U8) return launch_rerank_shape<K_U8>(a, st);
    if (dtype == JX_F16) return launch_rerank_shape<K_F16>(a, st);
    bool done = false;
    const hipError_t e = launch_rerank_sketch(a, st, &done);
    return e != hipSuccess || done ? e : launch_rerank_shape<K_F32>(a, st);
}

}  // namespace jx
