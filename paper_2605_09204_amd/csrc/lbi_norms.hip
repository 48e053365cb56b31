// Spectral and rank-normalised Frobenius norms of a stack of r x r matrices
// (gfx950): the interface-Jacobian statistics of the appendix "Interface
// Jacobian Structure" (local ||J_k||_2, suffix ||P_k||_2 = ||J_k^T ...
// J_{K-1}^T||_2, local ||J_k||_F / sqrt(r)).
//
// Per matrix M (fp32 or bf16 storage):
//  1. M is read once; m = max |M_ij| is reduced and Ms = M 2^-e, with
//     2^e <= m < 2^(e+1) (an exact scaling), is formed in registers.
//  2. H_0 = Ms Ms^T on the matrix cores.
//  3. Up to T times: H <- (H / tr H)(H / tr H).  H stays symmetric positive
//     semidefinite with every entry in [-1, 1]; after t steps it is a
//     multiple of (Ms Ms^T)^(2^t).  The steps end early once the trace of the
//     new H is at least 1 - d, d = 2^-8 (see below).
//  4. v = the row of H with the largest diagonal entry; the Rayleigh quotient
//     ||Ms^T v||^2 / ||v||^2 of Ms Ms^T gives sigma_1(M) = 2^e sqrt(quotient).
// A zero matrix gives 0 and 0; a matrix with a NaN or infinite entry NaN and NaN.
// Error of step 4 in exact arithmetic, with no spectral gap assumed: with
// x_k = sigma_k^2 / sigma_1^2 and weights c_k of v's row on the eigenvectors,
// 1 - quotient / sigma_1^2 <= max_x x^(2^T) (1 - x) / (row's diagonal)
// <= r / (exp(1) 2^T) (the diagonal is at least 1/r of the trace); T = 24
// puts it at 2.8e-6 for r = 128 (1.4e-6 for sigma).
// The early end: let u_k (sum 1) be the eigenvalues of the normalised H before
// a step.  The new trace is sum u_k^2 <= u_1, so a new trace of at least 1 - d
// means sum_{k>1} u_k <= d, and the new H has the eigenvalues u_k^2.  Its row v
// has c_1^2 u_1^2 >= 1/r - d^2 of its weight on the leading vector, so the
// quotient falls short by at most sum_{k>1} u_k^4 / (c_1^2 u_1^4), about
// r d^4 = 3e-8 at r = 128: below float32 rounding.  Spectra with a leading
// value 1.7 times the next end after five steps, 64 values drawn from
// U[0.9, 1.1] after about a dozen; equal leading values take all T.
//
// Products: every value is cut into three bf16 parts that sum to it exactly
// (split_pair) and the six partial products down to 2^-16 of the leading one
// run on the bf16 matrix cores with fp32 accumulation, as in the scan's fp32
// arithmetic.  These cost 6/16 of the fp32 matrix cores' cycles.
//
// H never leaves the registers (r <= 64, one wavefront per matrix, no
// barriers): the accumulator layout of v_mfma_f32_16x16x32 (lane l holds rows
// 16 I + 4 (l / 16) + v of column 16 N + l % 16) is the B operand layout for
// column block N with k taken in the order of the lane's rows, and, H being
// symmetric, also the A operand layout for row block N.  So the operands of a
// squaring are the split accumulators themselves.  At r = 128 four waves share
// a matrix, each holding two column blocks; the split operands of a k pair go
// round through LDS (24 KB, two buffers, one barrier per k pair).
// What bounds it: the matrix cores and the splits beside them (at r = 64 per
// squaring and wave 192 MFMAs of 16 cycles and about 290 VALU instructions).
// 8192 matrices at r = 64: 121 us with concentrated spectra, 312 us with
// U[0.9, 1.1]; with H in LDS, fp32 MFMAs and all T steps it was 842 us for
// both (r = 128, 4096 matrices: 448 and 1004 us against 3230).

#include "lbi_device.hpp"
#include "lbi_internal.h"

namespace lbi {
namespace {

constexpr int kThreads = 256;
constexpr int kSquarings = 24;
constexpr float kEndTrace = 1.0f - 1.0f / 256.0f;  // 1 - d of the early end

template <int R> struct NormGeo {
    static constexpr int WPM = R == 128 ? 4 : 1;  // waves per matrix
    static constexpr int MPW = 4 / WPM;           // matrices per workgroup
    static constexpr int NB = R / 16;             // 16-row blocks
    static constexpr int CB = NB / WPM;           // column blocks per wave
    static constexpr int NP = (NB + 1) / 2;       // k pairs (32 deep)
};

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        x += __shfl_xor(x, o);
    return x;
}

__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        x = fmaxf(x, __shfl_xor(x, o));
    return x;
}

// Four consecutive entries of a matrix in storage dtype, widened to fp32.
template <bool BF16> __device__ __forceinline__ f4 load4(const void *p, int64_t idx)
{
    if constexpr (BF16) {
        const u2 w = *(const u2 *)((const uint16_t *)p + idx);
        return f4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & kHighHalf),
                  __uint_as_float(w[1] << 16), __uint_as_float(w[1] & kHighHalf)};
    } else {
        return *(const f4 *)((const float *)p + idx);
    }
}

// Sum (or max) over the lanes of one matrix: the wave, or the workgroup
// through the four-float exchange area red (every lane gets the result).
template <int WPM, bool MAX>
__device__ __forceinline__ float matrix_reduce(float x, float *red)
{
    x = MAX ? wave_max(x) : wave_sum(x);
    if constexpr (WPM > 1) {
        const int w = threadIdx.x / 64;
        __syncthreads();  // red free (earlier readers done)
        if (threadIdx.x % 64 == 0)
            red[w] = x;
        __syncthreads();
        x = MAX ? fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))
                : (red[0] + red[1]) + (red[2] + red[3]);
    }
    return x;
}

// The three bf16 parts of one operand: 8 values per lane, k = 4 q + v of row
// blocks 2p (first four) and 2p + 1.
struct Parts {
    bf16x8 h, m, l;
};
__device__ __forceinline__ Parts split8(const f4 &a, const f4 &b)
{
    const Split2 s0 = split_pair(a[0], a[1]), s1 = split_pair(a[2], a[3]);
    const Split2 s2 = split_pair(b[0], b[1]), s3 = split_pair(b[2], b[3]);
    return {__builtin_bit_cast(bf16x8, u4{s0.h, s1.h, s2.h, s3.h}),
            __builtin_bit_cast(bf16x8, u4{s0.m, s1.m, s2.m, s3.m}),
            __builtin_bit_cast(bf16x8, u4{s0.l, s1.l, s2.l, s3.l})};
}

// H[i][t] (block rows 16 i, columns 16 (wm CB + t)) = sum over k of x(row, k)
// x(col, k), x given as scale * X[I][t] in the accumulator layout: element v of
// X[I][t] is x(16 (wm CB + t) + l % 16, 16 I + 4 (l / 16) + v).  X and H may be
// the same array.  r = 128: sx is the exchange area; every wave of the
// workgroup calls it the same number of times.
template <int R>
__device__ __forceinline__ void gram(f4 (&H)[NormGeo<R>::NB][NormGeo<R>::CB],
                                     const f4 (&X)[NormGeo<R>::NB][NormGeo<R>::CB], float scale,
                                     bf16x8 *sx)
{
    using G = NormGeo<R>;
    constexpr int NB = G::NB, CB = G::CB;
    const f4 zero = f4{0.0f, 0.0f, 0.0f, 0.0f};
    f4 acc[NB][CB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int t = 0; t < CB; ++t)
            acc[i][t] = zero;
#pragma unroll
    for (int p = 0; p < G::NP; ++p) {
        Parts o[CB];
#pragma unroll
        for (int t = 0; t < CB; ++t)
            o[t] = split8(X[2 * p][t] * scale, NB > 1 ? X[NB > 1 ? 2 * p + 1 : 0][t] * scale : zero);
        if constexpr (G::WPM == 1) {
            // the six partial products, each over all blocks in turn
#define LBI_NORM_TERM(A, B)                                                                   \
    _Pragma("unroll") for (int i = 0; i < NB; ++i)                                            \
        _Pragma("unroll") for (int t = 0; t < CB; ++t) acc[i][t] =                            \
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(o[i].A, o[t].B, acc[i][t], 0, 0, 0);
            LBI_NORM_TERM(h, h)
            LBI_NORM_TERM(h, m)
            LBI_NORM_TERM(m, h)
            LBI_NORM_TERM(h, l)
            LBI_NORM_TERM(l, h)
            LBI_NORM_TERM(m, m)
#undef LBI_NORM_TERM
        } else {
            // block i's operand sits at [p & 1][i][part][lane]; a buffer is
            // written again two k pairs later, past the barrier after its reads
            const int lane = threadIdx.x % 64, wm = threadIdx.x / 64;
            bf16x8 *buf = sx + (p & 1) * (NB * 3 * 64);
#pragma unroll
            for (int t = 0; t < CB; ++t) {
                bf16x8 *d = buf + (wm * CB + t) * 3 * 64 + lane;
                d[0] = o[t].h;
                d[64] = o[t].m;
                d[128] = o[t].l;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const bf16x8 *d = buf + i * 3 * 64 + lane;
                const bf16x8 ah = d[0], am = d[64], al = d[128];
#pragma unroll
                for (int t = 0; t < CB; ++t) {
                    f4 c = acc[i][t];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, o[t].h, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, o[t].m, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, o[t].h, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, o[t].l, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, o[t].h, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, o[t].m, c, 0, 0, 0);
                    acc[i][t] = c;
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int t = 0; t < CB; ++t)
            H[i][t] = acc[i][t];
}

template <int R, bool BF16>
__global__ __launch_bounds__(kThreads, 2) void norms_kernel(const void *M, int64_t n, float *spec,
                                                           float *fro)
{
    using G = NormGeo<R>;
    constexpr int NB = G::NB, CB = G::CB, WPM = G::WPM;
    __shared__ __attribute__((aligned(16))) float sv[G::MPW][R];  // the row v of each matrix
    __shared__ float red[4];
    __shared__ int redi[4];
    __shared__ __attribute__((aligned(16))) bf16x8 sx[WPM > 1 ? 2 * NB * 3 * 64 : 1];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int q = lane / 16, li = lane % 16;
    const int slot = wave / WPM;  // matrix within the workgroup
    const int wm = wave % WPM;    // wave within the matrix
    const int64_t g = (int64_t)blockIdx.x * G::MPW + slot;
    const bool live = g < n;
    const int64_t base = g * R * R;

    // 1. read M: H[I][t] = columns 16 I + 4 q .. + 3 of row 16 (wm CB + t) + li
    f4 H[NB][CB];
    float mx = 0.0f, poison = 0.0f;  // poison: NaN once any entry is not finite
#pragma unroll
    for (int t = 0; t < CB; ++t)
#pragma unroll
        for (int i = 0; i < NB; ++i)
            H[i][t] = live ? load4<BF16>(M, base + (16 * (wm * CB + t) + li) * R + 16 * i + 4 * q)
                           : f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < CB; ++t)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                mx = fmaxf(mx, fabsf(H[i][t][c]));
                poison += H[i][t][c] * 0.0f;
            }
    const float m = matrix_reduce<WPM, true>(mx, red);
    poison = matrix_reduce<WPM, false>(poison, red);
    // Ms = M 2^-e with 2^e <= m < 2^(e+1), scaled exactly in two halves (a
    // single factor would overflow for subnormal m)
    const int e = (m > 0.0f && m <= 3.0e38f) ? ilogbf(m) : 0;
    const float s1 = ldexpf(1.0f, -(e / 2)), s2 = ldexpf(1.0f, -(e - e / 2));
    // sum of Ms^2 (the Frobenius norm without overflow or underflow)
    float ssn = 0.0f;
#pragma unroll
    for (int t = 0; t < CB; ++t)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            H[i][t] = (H[i][t] * s1) * s2;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                ssn += H[i][t][c] * H[i][t][c];
        }
    const float fro2 = matrix_reduce<WPM, false>(ssn, red);
    if (fro && live && lane == 0 && wm == 0)
        fro[g] = ldexpf(sqrtf(fro2 / (float)R), e) + poison;
    if (!spec)
        return;

    // 2-3. H_0 = Ms Ms^T, then normalised squarings.  The diagonal entry of
    // column 16 (wm CB + t) + li sits in row block wm CB + t, lane group
    // q = li / 4, element li % 4.
    const bool dlane = q == li / 4;
    auto diag = [&](int t) {
        float d = 0.0f;
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (WPM == 1 ? i == t : i == wm * CB + t) {
                const f4 x = H[i][t];
                d = (li & 2) ? ((li & 1) ? x[3] : x[2]) : ((li & 1) ? x[1] : x[0]);
            }
        return d;
    };
    gram<R>(H, H, 1.0f, sx);
#pragma unroll 1
    for (int t = 0; t < kSquarings; ++t) {
        float d = 0.0f;
#pragma unroll
        for (int u = 0; u < CB; ++u)
            d += diag(u);
        // (the same in every lane of the matrix, so its waves end together)
        const float tr = matrix_reduce<WPM, false>(dlane ? d : 0.0f, red);
        if ((t > 0 && tr >= kEndTrace) || !(tr > 0.0f))
            break;
        gram<R>(H, H, 1.0f / tr, sx);
    }

    // 4. v = row i* of H (largest diagonal entry; the lowest index on ties)
    float best = -1.0f;
    int bi = 0;
#pragma unroll
    for (int t = 0; t < CB; ++t) {
        const float d = dlane ? diag(t) : -1.0f;
        if (d > best) {
            best = d;
            bi = 16 * (wm * CB + t) + li;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float ob = __shfl_xor(best, o);
        const int oi = __shfl_xor(bi, o);
        if (ob > best || (ob == best && oi < bi)) {
            best = ob;
            bi = oi;
        }
    }
    if constexpr (WPM > 1) {
        __syncthreads();
        if (lane == 0) {
            red[wm] = best;
            redi[wm] = bi;
        }
        __syncthreads();
        best = red[0];
        bi = redi[0];
#pragma unroll
        for (int u = 1; u < WPM; ++u)
            if (red[u] > best) {
                best = red[u];
                bi = redi[u];
            }
    }
    // (row i* is column i*: lanes li = i* % 16 of the wave that holds its block)
#pragma unroll
    for (int t = 0; t < CB; ++t)
        if (bi / 16 == wm * CB + t && li == bi % 16)
#pragma unroll
            for (int i = 0; i < NB; ++i)
                *(f4 *)&sv[slot][16 * i + 4 * q] = H[i][t];
    if constexpr (WPM > 1) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    const float *v = sv[slot];
    float vr[NB];  // v at rows 16 i + li
    float vv = 0.0f;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        vr[i] = v[16 * i + li];
        vv += vr[i] * vr[i];
    }
    vv = q == 0 ? vv : 0.0f;
    vv = wave_sum(vv);
    // w = Ms^T v over this wave's columns: row sums over li
    float w[4 * CB];
#pragma unroll
    for (int t = 0; t < CB; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            w[4 * t + c] = 0.0f;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int t = 0; t < CB; ++t) {
            f4 a = live ? load4<BF16>(M, base + (16 * i + li) * R + 16 * (wm * CB + t) + 4 * q)
                        : f4{0.0f, 0.0f, 0.0f, 0.0f};
            a = (a * s1) * s2;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                w[4 * t + c] += a[c] * vr[i];
        }
    // lane li ends with value li >> S; 2^S lanes share one, the first counts it
    constexpr int S = 2 - ilog2(CB);
    group_reduce<16, 4 * CB>(w, li);
    float ww = (li & ((1 << S) - 1)) == 0 ? w[0] * w[0] : 0.0f;
    ww = matrix_reduce<WPM, false>(ww, red);
    if (live && lane == 0 && wm == 0)
        spec[g] = (vv > 0.0f ? ldexpf(sqrtf(ww / vv), e) : 0.0f) + poison;
}

template <int R>
hipError_t norms_r(const void *M, bool bf16, int64_t n, float *spec, float *fro, hipStream_t st)
{
    using G = NormGeo<R>;
    const unsigned grid = (unsigned)((n + G::MPW - 1) / G::MPW);
    if (bf16)
        hipLaunchKernelGGL((norms_kernel<R, true>), dim3(grid), dim3(kThreads), 0, st, M, n, spec,
                           fro);
    else
        hipLaunchKernelGGL((norms_kernel<R, false>), dim3(grid), dim3(kThreads), 0, st, M, n, spec,
                           fro);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_norms(const void *M, bool bf16, int64_t n, int32_t r, float *spec, float *fro,
                        hipStream_t stream)
{
    switch (r) {
    case 16: return norms_r<16>(M, bf16, n, spec, fro, stream);
    case 32: return norms_r<32>(M, bf16, n, spec, fro, stream);
    case 64: return norms_r<64>(M, bf16, n, spec, fro, stream);
    default: return norms_r<128>(M, bf16, n, spec, fro, stream);
    }
}

}  // namespace lbi
