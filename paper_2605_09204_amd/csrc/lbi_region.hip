// Phase 1 of Algorithm "Bounded-Interface Backpropagation" (gfx950): the
// interface Jacobians J_k = dR_k(m_k) I_r (Eq. "jacobian-identity-
// construction") of the synthetic region map of Eq. "concrete-region-arch",
//
//   m_{k+1} = R_k(m_k) = LN(m_k + alpha_k Enc_k(pool(Phi_k(x_embed + Dec_k(m_k))))),
//   Dec_k(m) = W_d2 silu(W_d1 m + b_d1) + b_d2          (r -> D -> D)
//   Phi_k(x) = x + W2 silu(W1 x), token by token          (D -> X -> D)
//   pool     = mean over the L tokens of a sequence
//   Enc_k(p) = W_e2 silu(W_e1 p + b_e1) + b_e2          (D -> D -> r)
//   LN       = LayerNorm over the r features, gain gamma, shift beta, eps 1e-5,
//
// for every sequence b and region k at once, written as A[b][k] = J_k^T, the
// operand of the scan.
//
// The tangent of all r directions, taken exactly: Dec_k's differential
// Jdec = W_d2 diag(silu'(a)) W_d1 (D x r) is the same for every token, so
// through Phi_k and the mean pool
//   dp = Jdec + W2 diag(gbar) W1 Jdec,   gbar = mean_l silu'(W1 x_l),
// and p = mean_l x_embed + d + W2 sbar with sbar = mean_l silu(W1 x_l).  The
// per-token work is therefore one product H = X_in W1^T per sequence and region
// (L x D x X), whose epilogue reduces silu(H) and silu'(H) over the tokens; H
// never reaches memory.  The r directions then go through skinny products with
// N = B r (all sequences of a region at once) and the LayerNorm Jacobian
//   J = diag(gamma) / sigma (I - 11^T / r - zhat zhat^T / r) (I + alpha Jenc).
//
// Arithmetic: bf16 operands on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16)
// with fp32 accumulation; x_embed + d and the tangent intermediates are rounded
// to bf16 (round to nearest even) where they feed a product; every vector,
// reduction and the LayerNorm part are fp32.
//
// The per-token product uses H = x_embed W1^T + 1 (W1 d)^T: x_embed is the
// same bf16 operand for every region, and d enters in fp32 through the column
// vector W1 d, added in the epilogue.
//
// Launches (each line one; steps that do not need each other share a launch):
//   bmv a -> silu(a), silu'(a) | xpart: 64-token partial means of x_embed
//   bmv d = Dec_k(m) | p1: P1 = (diag(silu'(a)) W_d1)^T | xfin: mean_l x_embed
//   gemm Jdec^T | bmv cvec = W1 d
//   region_dma  per (k, 128 columns of X, part of the tokens, b): the token
//               product and its reductions
//   gemm U'^T = (W1 Jdec)^T scaled by gbar | bmv p = mean x_embed + d + W2 sbar
//   gemm dp^T | bmv e -> silu(e), silu'(e)
//   gemm T'^T | bmv Enc_k
//   gemm Jenc^T | ln_fwd: z = m + alpha Enc, LayerNorm -> m_{k+1}, zhat, 1/sigma
//   ln_jac: J, stored transposed as A[b][k]

#include <type_traits>

#include "lbi_device.hpp"
#include "lbi_internal.h"
#include "lbi_region_args.hpp"

namespace lbi {
namespace {

constexpr int kT = 256;
constexpr int BM = 128, BN = 128, BK = 64;
constexpr int TILE = 128 * BK;  // bf16 elements of one LDS tile (no padding)
constexpr float kLnEps = 1e-5f;

// Workgroup lists.  A launch dimension holds fewer than 2^32 work items (2^24
// workgroups of 256; past that the runtime refuses a launch, or starts what is left of
// the number modulo 2^32), so a list goes over rows of kGridRow workgroups, a multiple
// of 8 for the order over the XCDs.  Workgroups past the list do nothing.
constexpr int64_t kGridRow = 1 << 20;
dim3 list_grid(int64_t n)
{
    return n <= kGridRow ? dim3((unsigned)n)
                         : dim3((unsigned)kGridRow, (unsigned)((n + kGridRow - 1) / kGridRow));
}
__device__ __forceinline__ int64_t list_index()
{
    return (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
}

// The logistic function through the hardware reciprocal (1 ulp): it needs no
// correctly rounded division, and rcp(inf) = 0 keeps the saturated end exact.
__device__ __forceinline__ float sigm(float h) { return __builtin_amdgcn_rcpf(1.0f + __expf(-h)); }
__device__ __forceinline__ float silu(float h) { return h * sigm(h); }
__device__ __forceinline__ float dsilu(float h)
{
    const float s = sigm(h);
    return s * (1.0f + h * (1.0f - s));
}

__device__ __forceinline__ float bf(const __bf16 *p, int64_t i) { return (float)p[i]; }

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        x += __shfl_xor(x, o);
    return x;
}

// ---- the tile pipeline shared by both products ---------------------------------
// LDS tile layout: 128 rows of 64 bf16 (eight 16-byte chunks), two rows per
// 256-byte line, chunk q of row R at line R / 2, slot ((R & 1) 8 + q) ^ (R / 2 & 7).
// The 16 lanes that a b128 access serves together then touch 16 distinct
// slots (all 64 banks) both when they read one chunk of 16 consecutive rows
// (an MFMA operand) and when they write the 8 chunks of 2 consecutive rows.
__device__ __forceinline__ int lds_off(int row, int q)
{
    return (row >> 1) * 128 + ((((row & 1) << 3) + q) ^ ((row >> 1) & 7)) * 8;
}

// 128 rows x 64 k of a row-major bf16 matrix (row stride ld) from row0, k0;
// rows >= nrows read as zero.  Thread t loads chunks c = t + 256 i: row c / 8,
// chunk c % 8, at the per-lane byte offsets voff (tile_offsets).  One buffer
// resource per call starts at (row0, k0) and ends with the last valid row, so
// the lanes of missing rows fall outside it and read zero (no lane masks).
__device__ __forceinline__ void tile_offsets(uint32_t (&voff)[4], int ld)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = threadIdx.x + kT * i;
        voff[i] = (uint32_t)(((c >> 3) * ld + (c & 7) * 8) * 2);
    }
}

__device__ __forceinline__ void tile_load(u4 (&v)[4], const uint32_t (&voff)[4],
                                          const __bf16 *base, int64_t ld, int64_t row0,
                                          int64_t nrows, int k0)
{
    const int64_t left = nrows - row0;
    const int valid = left < 128 ? (int)left : 128;
    // the last valid row's chunks end at most 2 (ld - k0 - 64) bytes before
    // valid * ld * 2 - k0 * 2; the first missing row starts at or past it
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(base + row0 * ld + k0), 0, (int)(valid * (int)ld * 2 - k0 * 2), kBufferWord3);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[i], 0, 0);
}

__device__ __forceinline__ void tile_store(const u4 (&v)[4], __bf16 *s)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = threadIdx.x + kT * i;
        *(u4 *)(s + lds_off(c >> 3, c & 7)) = v[i];
    }
}

// ---- operands loaded straight into LDS ---------------------------------------------
typedef int i4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i4 dma_rsrc(const void *base, uint32_t bytes)
{
    // (the values are wave-uniform; the scalar registers an asm operand of
    // class "s" needs are made explicit)
    const uint64_t x = (uint64_t)(uintptr_t)base;
    i4 v;
    v[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    v[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(x >> 32) & 0xFFFFu));
    v[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    v[3] = kBufferWord3;
    return v;
}
// 16 bytes per lane from rs at voff + soff into LDS at lds + 16 lane; M0 (the
// LDS destination, one wait state after writing it) is saved and restored in
// the asm
__device__ __forceinline__ void dma_b128(uint32_t lds, i4 rs, int voff, int soff)
{
    uint32_t keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %2, %3, %4 offen lds\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep)
                 : "s"(lds), "v"(voff), "s"(rs), "s"(soff)
                 : "memory");
}
// all of this wave's loads but the N most recent, and its LDS operations, done;
// then the workgroup barrier (the waits are the compiler's own, so it counts
// them when it places its LDS waits)
template <int N> __device__ __forceinline__ void dma_barrier()
{
    __builtin_amdgcn_s_waitcnt((N & 15) | (((N >> 4) & 3) << 14) | (7 << 4));
    __builtin_amdgcn_s_barrier();
}

// this wave's loads done, and no memory operation moved over the wait
__device__ __forceinline__ void dma_wait()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((15) << 8 | (7 << 4));
    asm volatile("" ::: "memory");
}
// this wave's LDS operations done; then the workgroup barrier
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
    __builtin_amdgcn_s_barrier();
}

// acc += A_tile(128 x 64) B_tile(128 x 64)^T for this wave's 64 x 64 quarter
// (waves 2 x 2; acc[i][j] is the 16 x 16 block (i, j); lane l holds rows
// 4 (l / 16) + v, column l % 16 of it)
__device__ __forceinline__ void mma_bk(f4 (&acc)[4][4], const __bf16 *sA, const __bf16 *sB, int wm,
                                       int wn, int lane)
{
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        bf16x8 a[4], b[4];
        const int q = ks * 4 + (lane >> 4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            a[i] = *(const bf16x8 *)(sA + lds_off(wm * 64 + i * 16 + (lane & 15), q));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            b[j] = *(const bf16x8 *)(sB + lds_off(wn * 64 + j * 16 + (lane & 15), q));
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
}

// ---- bmv: y[b][k] = W[k] v[b][k] (+ bias[k]) (+ add1[b][k]) (+ add2[b][k]) -----
// for every sequence b of region k, fp32 sums of bf16 weights times fp32
// vectors; outputs y, silu(y) and silu'(y) (each optional).  A wave takes 8
// rows and NB sequences: each weight row is read once per region and NB
// sequences.  The workgroup's vectors go through LDS, kBmvCols / NB columns of
// each at a time, so that a step of a wave waits for its weights only.
struct BmvArgs {
    const __bf16 *W;
    int64_t sW;  // region stride (elements); rows N of C columns
    const float *v;  // the sum of nv vectors v_ss apart (nv 0: one)
    int64_t v_sb, v_sk;
    const float *bias;
    int64_t s_bias;
    const float *add1;
    int64_t a1_sb, a1_sk;
    const float *add2;
    int64_t a2_sb, a2_sk;
    float *y, *ys, *yd;
    int64_t y_sb, y_sk;
    int64_t B;
    int N, C;
    int nv = 0;
    int64_t v_ss = 0;
};

// Workgroups of a bmv over K regions (rows fastest, then regions, then groups
// of NB sequences).
__host__ __device__ __forceinline__ int64_t bmv_blocks(int N, int64_t K, int64_t B, int NB)
{
    return (int64_t)((N + 31) / 32) * K * ((B + NB - 1) / NB);
}

constexpr int kBmvCols = 8192;  // 32 KB of LDS
template <int NB>
__device__ __forceinline__ void bmv_block(const BmvArgs &a, int64_t K, int64_t blk, char *smem)
{
    static_assert(NB == 2 || NB == 8, "sequences per wave");
    const int nx = (a.N + 31) / 32;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t k = (blk / nx) % K, b0 = blk / nx / K * NB;
    const int n0 = (int)(blk % nx) * 32 + w * 8;
    const __bf16 *W = a.W + k * a.sW;
    constexpr int LIVE = 8 * NB;
    float acc[LIVE];  // [row rr][sequence bb]
#pragma unroll
    for (int i = 0; i < LIVE; ++i)
        acc[i] = 0.0f;
    constexpr int CH = kBmvCols / NB;
    float *sv = (float *)smem;  // [NB][CH]
    for (int c0 = 0; c0 < a.C; c0 += CH) {
        const int cn = a.C - c0 < CH ? a.C - c0 : CH;
        if (c0 > 0)
            __syncthreads();
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
            for (int c = 4 * threadIdx.x; c < cn; c += 4 * kT) {
                f4 x = f4{0.0f, 0.0f, 0.0f, 0.0f};
                if (b0 + bb < a.B) {
                    const float *vp = a.v + (b0 + bb) * a.v_sb + k * a.v_sk + c0 + c;
                    x = *(const f4 *)vp;
                    for (int u = 1; u < a.nv; ++u)
                        x += *(const f4 *)(vp + u * a.v_ss);
                }
                *(f4 *)&sv[bb * CH + c] = x;
            }
        __syncthreads();
#pragma unroll 2
        for (int c = lane * 8; c < cn; c += 64 * 8) {
            bf16x8 wv[8];
#pragma unroll
            for (int rr = 0; rr < 8; ++rr)
                wv[rr] = n0 + rr < a.N
                             ? *(const bf16x8 *)(W + (int64_t)(n0 + rr) * a.C + c0 + c)
                             : bf16x8{};
#pragma unroll
            for (int bb = 0; bb < NB; ++bb) {
                const f4 x0 = *(const f4 *)&sv[bb * CH + c], x1 = *(const f4 *)&sv[bb * CH + c + 4];
#pragma unroll
                for (int rr = 0; rr < 8; ++rr)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc[rr * NB + bb] += (float)wv[rr][e] * (e < 4 ? x0[e & 3] : x1[e & 3]);
            }
        }
    }
    // the LIVE partial sums over the 64 lanes: the first lane of each 64 / LIVE
    // ends with one of them
    {
        const bool upper = (lane >> 5) & 1;
        float q[LIVE / 2];
#pragma unroll
        for (int i = 0; i < LIVE / 2; ++i) {
            const float keep = upper ? acc[i + LIVE / 2] : acc[i];
            const float send = upper ? acc[i] : acc[i + LIVE / 2];
            q[i] = keep + __shfl_xor(send, 32);
        }
        group_reduce<32, LIVE / 2>(q, lane & 31);
        acc[0] = q[0];
    }
    constexpr int SH = 5 - ilog2(LIVE / 2);
    const int idx = (lane >> 5) * (LIVE / 2) + ((lane & 31) >> SH);
    const int rr = idx / NB, bb = idx % NB;
    const int n = n0 + rr;
    const int64_t b = b0 + bb;
    if ((lane & ((1 << SH) - 1)) == 0 && n < a.N && b < a.B) {
        float y = acc[0];
        if (a.bias)
            y += a.bias[k * a.s_bias + n];
        if (a.add1)
            y += a.add1[b * a.a1_sb + k * a.a1_sk + n];
        if (a.add2)
            y += a.add2[b * a.a2_sb + k * a.a2_sk + n];
        const int64_t o = b * a.y_sb + k * a.y_sk + n;
        if (a.y)
            a.y[o] = y;
        if (a.ys)
            a.ys[o] = silu(y);
        if (a.yd)
            a.yd[o] = dsilu(y);
    }
}

// ---- p1: P1[k][b r + j][h] = W_d1[k][h][j] silu'(a)[b][k][h], the A operand of
//      Jdec^T; 64 values of h per workgroup, transposed through LDS so that
//      both the reads of W_d1 rows and the writes of P1 rows are contiguous
__device__ __forceinline__ void p1_block(const RegionArgs &q, int64_t blk, char *smem)
{
    float(*tile)[129] = (float(*)[129])smem;  // [h - h0][j], r <= 128
    const int64_t bk = blk % (q.B * q.K), b = bk / q.K, k = bk % q.K;
    const int D = q.D, r = q.r;
    const int h0 = (int)(blk / (q.B * q.K)) * 64;
    const __bf16 *Wd1 = (const __bf16 *)q.W_d1 + k * (int64_t)D * r;
    const float *sa = q.sa + bk * D;
    for (int idx = threadIdx.x; idx < 64 * r; idx += kT) {
        const int hh = idx / r, j = idx % r;
        tile[hh][j] = bf(Wd1, (int64_t)(h0 + hh) * r + j) * sa[h0 + hh];
    }
    __syncthreads();
    __bf16 *P1 = q.P1 + (k * q.B + b) * (int64_t)r * D;
    for (int idx = threadIdx.x; idx < 64 * r; idx += kT) {
        const int j = idx / 64, hh = idx % 64;
        P1[(int64_t)j * D + h0 + hh] = (__bf16)tile[hh][j];
    }
}

// ---- xpart / xfin: mean over the tokens of x_embed, 64-token partial sums first
__device__ __forceinline__ void xpart_block(const RegionArgs &q, int64_t blk)
{
    // thread t sums the 8 columns 8t .. 8t + 7 over the workgroup's 64 tokens
    const int64_t nch = (q.L + 63) / 64, b = blk / nch, ch = blk % nch;
    const int64_t l0 = ch * 64, l1 = l0 + 64 < q.L ? l0 + 64 : q.L;
    const int c = threadIdx.x * 8;
    if (c >= q.D)
        return;
    const __bf16 *x = (const __bf16 *)q.x_embed + b * q.L * q.D + c;
    float s[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    // (unrolled: eight token loads in flight rather than one)
#pragma unroll 8
    for (int64_t l = l0; l < l1; ++l) {
        const bf16x8 v = *(const bf16x8 *)(x + l * q.D);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            s[e] += (float)v[e];
    }
    float *o = q.xpart + (b * nch + ch) * q.D + c;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        o[e] = s[e];
}

__device__ __forceinline__ void xfin_block(const RegionArgs &q, int64_t blk)
{
    const int64_t b = blk % q.B;
    const int c = (int)(blk / q.B) * kT + threadIdx.x;
    if (c >= q.D)
        return;
    const int64_t nch = (q.L + 63) / 64;
    float s = 0.0f;
#pragma unroll 8
    for (int64_t ch = 0; ch < nch; ++ch)
        s += q.xpart[(b * nch + ch) * q.D + c];
    q.xbar[b * q.D + c] = s / (float)q.L;
}

// ---- region_dma: sbar, gbar for 128 columns of X, one sequence and region -----
// H = x_embed[b] W1[k]^T + 1 cvec[b, k]^T (cvec = W1 d) over all L tokens in
// 128-row tiles; the epilogue of each tile adds silu(H) and silu'(H) of its
// valid rows into per-lane column sums.  Both operands load straight into LDS
// (buffer_load_dwordx4 ... lds, the row layout of lds_off): 128 x 128 tiles,
// four waves of 64 x 64, two 64-deep stages (64 KB, two workgroups per CU), one
// pipeline over (row tile, k block), so that a tile's epilogue runs while the
// next tile's first stage loads.
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(2, 2))) void region_dma_kernel(
    RegionArgs q)
{
    constexpr int OP = BM * BK * 2;   // bytes of one operand's stage (16 KB)
    constexpr int STG = 2 * OP;
    constexpr int NL = OP / 1024 / 4; // 1 KB loads per wave, operand and stage
    __shared__ __attribute__((aligned(1024))) char smem[2 * STG];
    __shared__ float sred[2][2][BN];
    typedef __attribute__((address_space(3))) char lchar;
    const uint32_t lbase = (uint32_t)(uintptr_t)(lchar *)smem;
    const int nxt = q.X / BN;
    const int64_t G = q.K * q.B * nxt * q.nsplit;
    int64_t lg = list_index();
    if (lg >= G)
        return;
    if (G % 8 == 0)
        lg = (lg % 8) * (G / 8) + lg / 8;
    // (this workgroup's row tiles: t0 .. t0 + ntile - 1, part sp of q.nsplit)
    const int64_t b = lg % q.B;
    const int sp = (int)((lg / q.B) % q.nsplit);
    const int64_t xt = (lg / (q.B * q.nsplit)) % nxt;
    const int64_t k = lg / (q.B * q.nsplit * nxt);
    const int ntl = (int)((q.L + BM - 1) / BM), per = (ntl + q.nsplit - 1) / q.nsplit;
    const int t0 = sp * per;
    const int ntile = t0 + per < ntl ? per : (ntl > t0 ? ntl - t0 : 0);
    const int D = q.D;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
    const int64_t bk = b * q.K + k;
    const __bf16 *Xe = (const __bf16 *)q.x_embed + b * q.L * D;
    const i4 rsB = dma_rsrc((const __bf16 *)q.W1 + (k * q.X + xt * BN) * (int64_t)D,
                            (uint32_t)BN * D * 2);
    float cv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        cv[j] = q.cvec[bk * q.X + xt * BN + wn * 64 + j * 16 + (lane & 15)];
    const int nk = D / BK;
    const int nstep = ntile * nk;
    // load d of a wave: rows 8 d' .. 8 d' + 7 (d' = w + 4 d) of a tile, lane ->
    // line rp = 4 d' + lane / 16, row 2 rp + (lane & 15) / 8, chunk (lane & 7) ^ (rp & 7)
    int vo[NL];
#pragma unroll
    for (int d = 0; d < NL; ++d) {
        const int rp = 4 * (w + 4 * d) + (lane >> 4);
        vo[d] = (2 * rp + ((lane & 15) >> 3)) * D * 2 + (((lane & 7) ^ (rp & 7)) << 4);
    }
    auto issue = [&](int s) {
        const int t = s / nk, kb = s - t * nk;
        const int64_t row0 = (int64_t)(t0 + t) * BM;
        const int vA = q.L - row0 < BM ? (int)(q.L - row0) : BM;
        const i4 rsA = dma_rsrc(Xe + row0 * D, (uint32_t)vA * D * 2);
        const uint32_t st = lbase + (uint32_t)((s & 1) * STG);
#pragma unroll
        for (int d = 0; d < NL; ++d) {
            const uint32_t blk = (uint32_t)((w + 4 * d) * 1024);
            dma_b128(__builtin_amdgcn_readfirstlane(st + blk), rsA, vo[d], kb * BK * 2);
            dma_b128(__builtin_amdgcn_readfirstlane(st + OP + blk), rsB, vo[d], kb * BK * 2);
        }
    };
    uint32_t ro[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        ro[ks] = (uint32_t)(lds_off(lane & 15, 4 * ks + (lane >> 4)) * 2);
    // column sums of s = sigmoid(h), silu(h) = h s and silu(h) s
    float s1[4] = {0.0f, 0.0f, 0.0f, 0.0f}, s2[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float s3[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    f4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    if (nstep > 0)
        issue(0);
    for (int s = 0; s < nstep; ++s) {
        dma_barrier<0>();  // stage s complete; stage s - 1 read by every wave
        if (s + 1 < nstep)
            issue(s + 1);
        const uint32_t st = lbase + (uint32_t)((s & 1) * STG);
        bf16x8 a[2][4], bb[2][4];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[ks][i] = *(const bf16x8 *)(lchar *)(uintptr_t)(st + ro[ks] +
                                                                  (wm * 64 + i * 16) * 128);
                bb[ks][i] = *(const bf16x8 *)(lchar *)(uintptr_t)(st + OP + ro[ks] +
                                                                   (wn * 64 + i * 16) * 128);
            }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], bb[ks][j],
                                                                         acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 32, 0);
        const int t = s / nk;
        if (s - t * nk == nk - 1) {
            // epilogue of row tile t over its valid rows (selects: rows past L
            // may hold anything); with s = sigmoid(h), silu = h s and
            // silu' = s + silu - silu s, the sums of s, silu and silu s carry
            // both reductions
            const int64_t rbase = (int64_t)(t0 + t) * BM + wm * 64 + 4 * (lane >> 4);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool ok = rbase + i * 16 + v < q.L;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float h = acc[i][j][v] + cv[j];
                        const float sg = sigm(h);
                        const float sl = h * sg;
                        s1[j] += ok ? sg : 0.0f;
                        s2[j] += ok ? sl : 0.0f;
                        s3[j] += ok ? sl * sg : 0.0f;
                    }
                }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    // lanes l, l ^ 16, l ^ 32, l ^ 48 hold the same columns; then the two
    // waves of a column half through LDS
    float cs[4], cg[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        cs[j] = s2[j];
        cg[j] = s1[j] + s2[j] - s3[j];
        cs[j] += __shfl_xor(cs[j], 16);
        cs[j] += __shfl_xor(cs[j], 32);
        cg[j] += __shfl_xor(cg[j], 16);
        cg[j] += __shfl_xor(cg[j], 32);
    }
    if (lane < 16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sred[0][wm][wn * 64 + j * 16 + lane] = cs[j];
            sred[1][wm][wn * 64 + j * 16 + lane] = cg[j];
        }
    }
    __syncthreads();
    if (tid < BN) {
        const float inv = 1.0f / (float)q.L;
        const int64_t o = (sp * q.B * q.K + bk) * q.X + xt * BN + tid;
        q.sbar[o] = (sred[0][0][tid] + sred[0][1][tid]) * inv;
        q.gbar[o] = (sred[1][0][tid] + sred[1][1][tid]) * inv;
    }
}

// ---- ln_fwd: z = m + alpha Enc, LayerNorm -> m_{k+1}, zhat, 1/sigma ------------
__device__ __forceinline__ void ln_fwd_wave(const RegionArgs &q, int64_t bk)
{
    const int r = q.r, lane = threadIdx.x & 63;
    const int64_t k = bk % q.K;
    const float alpha = q.alpha[k];
    float z[2];
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + 64 * u;
        z[u] = i < r ? q.m[bk * r + i] + alpha * q.encv[bk * r + i] : 0.0f;
        s += z[u];
    }
    const float mu = wave_sum(s) / (float)r;
    float v = 0.0f;
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (lane + 64 * u < r)
            v += (z[u] - mu) * (z[u] - mu);
    const float is = 1.0f / sqrtf(wave_sum(v) / (float)r + kLnEps);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + 64 * u;
        if (i < r) {
            const float zh = (z[u] - mu) * is;
            q.zhat[bk * r + i] = zh;
            if (q.m_next)
                q.m_next[bk * r + i] = q.gamma[k * r + i] * zh + q.beta[k * r + i];
        }
    }
    if (lane == 0)
        q.isig[bk] = is;
}

// ---- gemm_nt: C[M][N] = A[M][K] B[N][K]^T per batch, with the epilogue
//      v = acc * scale[batch][row >> grp_shift][col] + add[batch][row][col] ------
struct GemmOp {
    const __bf16 *A;
    int64_t lda, sA;
    const __bf16 *B;
    int64_t ldb, sB;
    void *C;
    int64_t ldc, sC;
    int64_t M, N;
    int K;
    const float *scale;  // NULL: 1; the sum of nscale arrays scale_ss apart (0: one)
    int64_t s_scale_b, s_scale_g;
    int grp_shift;  // rows per scale row: 2^grp_shift (1, or the interface width)
    const __bf16 *add;  // NULL: 0 (ld ldc, batch stride sC)
    bool out_bf16;
    // B's batch index is (bz0 + z) / bdiv (bdiv 0: z), so that a batch of
    // (sequence, region) pairs ordered region-major takes its region's weights
    int64_t bz0 = 0, bdiv = 0;
    // act: C = silu(v) (bf16) and C2 = silu'(v) (fp32, same index) in place of v
    bool act = false;
    float *C2 = nullptr;
    int nscale = 0;
    int64_t scale_ss = 0;
};

// The epilogue of a wave's NI x NJ blocks from (row0, col0).  Every load comes
// before the first store (which the compiler could not move them across), so
// that they take one latency.  A 16-row block has one scale row: grp_shift >= 4.
template <int NI, int NJ>
__device__ __forceinline__ void gemm_out(const GemmOp &g, int64_t z, int64_t row0, int64_t col0,
                                         f4 (&acc)[NI][NJ])
{
    const int lane = threadIdx.x & 63, q = lane >> 4, li = lane & 15;
    if (g.scale) {
        float f[NI][NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                f[i][j] = 0.0f;
        int u = 0;
        do {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int64_t row = row0 + 16 * i, col = col0 + 16 * j + li;
                    if (row < g.M && col < g.N)
                        f[i][j] += g.scale[z * g.s_scale_b + (row >> g.grp_shift) * g.s_scale_g +
                                           col + u * g.scale_ss];
                }
        } while (++u < g.nscale);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[i][j][v] *= f[i][j];
    }
    if (g.add) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int64_t row = row0 + 16 * i + 4 * q + v, col = col0 + 16 * j + li;
                    if (row < g.M && col < g.N)
                        acc[i][j][v] += (float)g.add[z * g.sC + row * g.ldc + col];
                }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = row0 + 16 * i + 4 * q + v;
            if (row >= g.M)
                continue;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int64_t col = col0 + 16 * j + li;
                if (col >= g.N)
                    continue;
                const int64_t o = z * g.sC + row * g.ldc + col;
                const float val = acc[i][j][v];
                if (g.act) {
                    ((__bf16 *)g.C)[o] = (__bf16)silu(val);
                    g.C2[o] = dsilu(val);
                } else if (g.out_bf16) {
                    ((__bf16 *)g.C)[o] = (__bf16)val;
                } else {
                    ((float *)g.C)[o] = val;
                }
            }
        }
}

// 128 x 128 tiles: tile (tn, tm) of batch z; smem 64 KB
__device__ __forceinline__ void gemm128_block(const GemmOp &g, int64_t tn, int64_t tm, int64_t z,
                                              char *smem)
{
    __bf16(*sA)[TILE] = (__bf16(*)[TILE])smem;
    __bf16(*sB)[TILE] = (__bf16(*)[TILE])(smem + 2 * TILE * sizeof(__bf16));
    const int64_t m0 = tm * BM, n0 = tn * BN;
    const __bf16 *A = g.A + z * g.sA;
    const __bf16 *B = g.B + (g.bdiv ? (g.bz0 + z) / g.bdiv : z) * g.sB;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wm = w >> 1, wn = w & 1;
    f4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const int nk = g.K / BK;
    int lkb = 0;  // next k block to load (two ahead of the products)
    uint32_t voa[4], vob[4];
    tile_offsets(voa, (int)g.lda);
    tile_offsets(vob, (int)g.ldb);
    auto load = [&](u4 (&va)[4], u4 (&vb)[4]) {
        if (lkb < nk) {
            tile_load(va, voa, A, g.lda, m0, g.M, lkb * BK);
            tile_load(vb, vob, B, g.ldb, n0, g.N, lkb * BK);
        }
        ++lkb;
    };
    u4 ra0[4], rb0[4], ra1[4], rb1[4];
    load(ra0, rb0);
    tile_store(ra0, sA[0]);
    tile_store(rb0, sB[0]);
    load(ra0, rb0);
    load(ra1, rb1);
    __syncthreads();
    int kb = 0, cur = 0;
    auto body = [&](u4 (&va)[4], u4 (&vb)[4]) -> bool {
        mma_bk(acc, sA[cur], sB[cur], wm, wn, lane);
        if (++kb == nk)
            return false;
        tile_store(va, sA[cur ^ 1]);
        tile_store(vb, sB[cur ^ 1]);
        __syncthreads();
        cur ^= 1;
        load(va, vb);
        return true;
    };
    for (;;) {
        if (!body(ra0, rb0))
            break;
        if (!body(ra1, rb1))
            break;
    }
    gemm_out(g, z, m0 + wm * 64, n0 + wn * 64, acc);
}

// TM x 64 tiles (TM 64 or 32) for products too small to fill the GPU with 128 x
// 128 ones: four waves of TM / 2 x 32, operands straight into LDS (dma_b128,
// the row layout of lds_off), a ring of four 64-deep stages with three in
// flight.  At this size a step is a few hundred cycles of products against a
// load latency of one to two thousand, so what counts is workgroups and bytes
// in flight.
constexpr int kGSt = 4;            // stages
constexpr int kGOp = 64 * BK * 2;  // bytes of the 64-row operand's stage (8 KB)
template <int TM> constexpr int gemm_small_lds() { return kGSt * (kGOp + TM * BK * 2); }
template <int TM>
__device__ __forceinline__ void gemm_small_block(const GemmOp &g, int64_t tn, int64_t tm, int64_t z,
                                                 char *smem)
{
    typedef __attribute__((address_space(3))) char lchar;
    constexpr int NI = TM / 32;            // 16-row blocks per wave
    constexpr int OPA = TM * BK * 2;       // bytes of A's stage
    constexpr int NLA = OPA / 1024 / 4;    // 1 KB loads per wave and stage: A,
    constexpr int NLB = kGOp / 1024 / 4;   // B
    constexpr int NL = NLA + NLB;
    const uint32_t lbase = (uint32_t)(uintptr_t)(lchar *)smem;
    const int64_t m0 = tm * TM, n0 = tn * 64;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w >> 1, wn = w & 1;
    const int vA = g.M - m0 < TM ? (int)(g.M - m0) : TM, vB = g.N - n0 < 64 ? (int)(g.N - n0) : 64;
    const int lda = (int)g.lda, ldb = (int)g.ldb;
    const i4 rsA = dma_rsrc(g.A + z * g.sA + m0 * g.lda, (uint32_t)(vA * lda * 2));
    const i4 rsB = dma_rsrc(g.B + (g.bdiv ? (g.bz0 + z) / g.bdiv : z) * g.sB + n0 * g.ldb,
                            (uint32_t)(vB * ldb * 2));
    // load d of a wave: rows 8 d' .. 8 d' + 7 (d' = w + 4 d) of an operand, lane ->
    // line rp = 4 d' + lane / 16, row 2 rp + (lane & 15) / 8, chunk (lane & 7) ^ (rp & 7)
    int voA[NLA], voB[NLB];
#pragma unroll
    for (int d = 0; d < NLB; ++d) {
        const int rp = 4 * (w + 4 * d) + (lane >> 4), row = 2 * rp + ((lane & 15) >> 3);
        const int ch = ((lane & 7) ^ (rp & 7)) << 4;
        if (d < NLA)
            voA[d < NLA ? d : 0] = row * lda * 2 + ch;
        voB[d] = row * ldb * 2 + ch;
    }
    const int nk = g.K / BK;
    auto issue = [&](int s) {
        const uint32_t st = lbase + (uint32_t)((s % kGSt) * (kGOp + OPA));
#pragma unroll
        for (int d = 0; d < NLB; ++d) {
            const uint32_t blk = (uint32_t)((w + 4 * d) * 1024);
            if (d < NLA)
                dma_b128(__builtin_amdgcn_readfirstlane(st + blk), rsA, voA[d < NLA ? d : 0],
                         s * BK * 2);
            dma_b128(__builtin_amdgcn_readfirstlane(st + OPA + blk), rsB, voB[d], s * BK * 2);
        }
    };
    f4 acc[NI][2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < kGSt - 1; ++s)
        if (s < nk)
            issue(s);
    uint32_t ro[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        ro[ks] = (uint32_t)(lds_off(lane & 15, 4 * ks + (lane >> 4)) * 2);
    for (int s = 0; s < nk; ++s) {
        // stage s complete (at most the two after it in flight), and stage
        // s - 1, whose place stage s + 3 takes, read by every wave
        if (s + 2 < nk)
            dma_barrier<2 * NL>();
        else if (s + 1 < nk)
            dma_barrier<NL>();
        else
            dma_barrier<0>();
        if (s + kGSt - 1 < nk)
            issue(s + kGSt - 1);
        const uint32_t st = lbase + (uint32_t)((s % kGSt) * (kGOp + OPA));
        bf16x8 a[2][NI], b[2][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
                a[ks][i] = *(const bf16x8 *)(lchar *)(uintptr_t)(st + ro[ks] +
                                                                  (wm * (TM / 2) + i * 16) * 128);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                b[ks][j] = *(const bf16x8 *)(lchar *)(uintptr_t)(st + OPA + ro[ks] +
                                                                  (wn * 32 + j * 16) * 128);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], b[ks][j],
                                                                         acc[i][j], 0, 0, 0);
    }
    gemm_out(g, z, m0 + wm * (TM / 2), n0 + wn * 32, acc);
}

// The tiles of a product, by their rows TM (128 x 128, 64 x 64, 32 x 64):
// columns fastest, then rows, then the batch.  Workgroup i runs on XCD i % 8
// (the workgroups before a product's in its launch are a multiple of 8), and
// each XCD takes one range of tiles, so that a region's weights go to one L2:
// dealt out one by one, the tiles that share a weight tile sat on different
// XCDs, and each read it from beyond its L2.
constexpr int tile_cols(int TM) { return TM == 128 ? 128 : 64; }
__host__ __device__ __forceinline__ int64_t gemm_tiles(const GemmOp &g, int64_t batch, int TM)
{
    const int TN = tile_cols(TM);
    return (g.N + TN - 1) / TN * ((g.M + TM - 1) / TM) * batch;
}
int64_t round8(int64_t n) { return (n + 7) / 8 * 8; }
int64_t gemm_blocks(const GemmOp &g, int64_t batch, int TM)
{
    return round8(gemm_tiles(g, batch, TM));
}
template <int TM>
__device__ __forceinline__ void gemm_block(const GemmOp &g, int64_t batch, int64_t i, char *smem)
{
    constexpr int TN = tile_cols(TM);
    const int64_t ntn = (g.N + TN - 1) / TN, ntm = (g.M + TM - 1) / TM;
    const int64_t n = gemm_tiles(g, batch, TM), blk = i % 8 * ((n + 7) / 8) + i / 8;
    if (i / 8 >= (n + 7) / 8 || blk >= n)
        return;
    const int64_t tn = blk % ntn, tm = blk / ntn % ntm, z = blk / ntn / ntm;
    if constexpr (TM == 128)
        gemm128_block(g, tn, tm, z, smem);
    else
        gemm_small_block<TM>(g, tn, tm, z, smem);
}
template <int TM> constexpr int gemm_lds()
{
    return TM == 128 ? 4 * TILE * 2 : gemm_small_lds<TM>();
}

template <int TM> __global__ __launch_bounds__(kT) void gemm_nt_kernel(GemmOp g, int64_t batch)
{
    __shared__ __attribute__((aligned(1024))) char smem[gemm_lds<TM>()];
    gemm_block<TM>(g, batch, list_index(), smem);
}

// ---- launches that join independent steps ------------------------------------------
// A step of the small ones takes 5 to 10 us, most of it latency, and two that
// do not need each other take as long together (19 launches became 9).

// in: a = W_d1 m (bmv), and the 64-token partial sums of x_embed
template <int NB>
__global__ __launch_bounds__(kT) void in_kernel(RegionArgs q, BmvArgs v, int64_t nb)
{
    __shared__ __attribute__((aligned(16))) char smem[kBmvCols * 4];
    const int64_t i = list_index();
    if (i < nb)
        bmv_block<NB>(v, q.K, i, smem);
    else if (i - nb < (q.L + 63) / 64 * q.B)
        xpart_block(q, i - nb);
}

// dec: d (bmv), P1, and the token mean of x_embed
template <int NB>
__global__ __launch_bounds__(kT) void dec_kernel(RegionArgs q, BmvArgs v, int64_t nb, int64_t np)
{
    __shared__ __attribute__((aligned(16))) char smem[64 * 129 * 4];
    const int64_t i = list_index();
    if (i < nb)
        bmv_block<NB>(v, q.K, i, smem);
    else if (i < nb + np)
        p1_block(q, i - nb, smem);
    else
        xfin_block(q, i - nb - np);
}

// a bmv and a product
template <int NB, int TM>
__global__ __launch_bounds__(kT) void gemm_bmv_kernel(GemmOp g, BmvArgs v, int64_t nb, int64_t K)
{
    __shared__ __attribute__((aligned(1024))) char smem[gemm_lds<TM>()];
    // (nb is rounded up to a multiple of 8)
    const int64_t i = list_index();
    if (i >= nb)
        gemm_block<TM>(g, K, i - nb, smem);
    else if (i < bmv_blocks(v.N, K, v.B, NB))
        bmv_block<NB>(v, K, i, smem);
}

// a product and the LayerNorm of the forward, a wave per (sequence, region)
template <int TM>
__global__ __launch_bounds__(kT) void gemm_ln_kernel(GemmOp g, int64_t ng, RegionArgs q)
{
    __shared__ __attribute__((aligned(1024))) char smem[gemm_lds<TM>()];
    const int64_t i = list_index();
    if (i < ng) {
        gemm_block<TM>(g, q.K, i, smem);
    } else {
        const int64_t bk = (i - ng) * 4 + threadIdx.x / 64;
        if (bk < q.B * q.K)
            ln_fwd_wave(q, bk);
    }
}

// ---- ln_jac: J = diag(gamma) / sigma (I - 11^T/r - zhat zhat^T/r)(I + alpha Jenc),
//      stored as A[b][k] = J^T ------------------------------------------------------
__global__ __launch_bounds__(kT) void ln_jac_kernel(RegionArgs q)
{
    extern __shared__ float lsh[];
    const int r = q.r;
    float *cm = lsh;    // [r] column means of dz
    float *cd = cm + r; // [r] column dots of dz with zhat, over r
    float *zh = cd + r; // [r]
    const int64_t bk = blockIdx.x, b = bk / q.K, k = bk % q.K;
    const float alpha = q.alpha[k];
    // Jenc^T[k][b r + j][i] = Jenc[i][j]; dz = I + alpha Jenc
    const float *JT = q.JencT + (k * q.B + b) * (int64_t)r * r;
    for (int i = threadIdx.x; i < r; i += kT)
        zh[i] = q.zhat[bk * r + i];
    __syncthreads();
    // kT / r lanes per column j of dz, each r^2 / kT of its rows
    const int tpr = kT / r, cpr = r / tpr;
    const int jc = threadIdx.x / tpr, i0 = (threadIdx.x % tpr) * cpr;
    float s = 0.0f, t = 0.0f;
#pragma unroll 4
    for (int e = 0; e < cpr; ++e) {
        const int i = i0 + e;
        const float v = (i == jc ? 1.0f : 0.0f) + alpha * JT[(int64_t)jc * r + i];
        s += v;
        t += zh[i] * v;
    }
    for (int o = 1; o < tpr; o <<= 1) {
        s += __shfl_xor(s, o);
        t += __shfl_xor(t, o);
    }
    if (i0 == 0) {
        cm[jc] = s / (float)r;
        cd[jc] = t / (float)r;
    }
    __syncthreads();
    const float is = q.isig[bk];
    float *A = q.A + bk * (int64_t)r * r;
    for (int idx = threadIdx.x; idx < r * r; idx += kT) {
        const int j = idx / r, i = idx % r;
        const float v = (i == j ? 1.0f : 0.0f) + alpha * JT[idx];
        A[idx] = q.gamma[k * r + i] * is * (v - cm[j] - zh[i] * cd[j]);
    }
}


// ==== the token-mixing block ======================================================
// Phi_k(x)_l = x_l + (W2 silu(W1 s_l)) silu(s_l) with the causal recurrence
// s_l = a_k s_{l-1} + (1 - a_k) x_l over the tokens (s_0 = 0).  The tangent of
// all r directions goes through every token: with Jdec (D x r) the same for
// each token, the state's tangent is c_l Jdec, c_l = 1 - a^l (the state of a
// constant input), and
//   dp = Jdec (1 + w) + (1/L) sum_l diag(silu(s_l)) W2 diag(silu'(W1 s_l)) W1 (c_l Jdec),
//   w  = mean_l y_l silu'(s_l) c_l,   y_l = W2 silu(W1 s_l),
// two products of r times the size of the forward's token products per
// sequence and region (Eq. "jacobian-work"), which nothing here shortcuts.

constexpr int64_t kCUs = 256;  // workgroups of the two tangent products: one per CU
constexpr int kSsmChunks = 8;  // token chunks per channel in the recurrence kernels

// ---- ssm_fwd: s (bf16, fp32) and c for 64 channels of one pair -------------------
// Thread (channel cc, chunk ch) runs its chunk of tokens from a zero state,
// then again from the state the chunks before it leave (a chunk of n tokens
// maps a state S to a^n S + its zero-start end state).
__global__ __launch_bounds__(64 * kSsmChunks) void ssm_fwd_kernel(RegionArgs q, int64_t p0)
{
    __shared__ float endS[kSsmChunks][64], endP[kSsmChunks][64];
    const int64_t z = blockIdx.y, pr = p0 + z, k = pr / q.B, b = pr % q.B;
    const int cc = threadIdx.x & 63, ch = threadIdx.x >> 6;
    const int dch = blockIdx.x * 64 + cc;  // D is a multiple of 64
    const int D = q.D;
    const int64_t L = q.L;
    const float a = q.decay[k * D + dch];
    const float ia = 1.0f - a;
    const float dv = q.d[(b * q.K + k) * D + dch];
    const int64_t per = (L + kSsmChunks - 1) / kSsmChunks;
    const int64_t l0 = ch * per < L ? ch * per : L;
    const int64_t l1 = l0 + per < L ? l0 + per : L;
    const __bf16 *x = (const __bf16 *)q.x_embed + b * L * D + dch;
    float st = 0.0f, pw = 1.0f;
#pragma unroll 8
    for (int64_t l = l0; l < l1; ++l) {
        st = a * st + ia * ((float)x[l * D] + dv);
        pw *= a;
    }
    endS[ch][cc] = st;
    endP[ch][cc] = pw;
    __syncthreads();
    float cs = 0.0f, cc1 = 0.0f;  // states entering the chunk: of x, of the constant 1
    for (int u = 0; u < ch; ++u) {
        cs = cs * endP[u][cc] + endS[u][cc];
        cc1 = cc1 * endP[u][cc] + (1.0f - endP[u][cc]);
    }
    const int64_t o = z * L * D + dch;
#pragma unroll 8
    for (int64_t l = l0; l < l1; ++l) {
        cs = a * cs + ia * ((float)x[l * D] + dv);
        cc1 = a * cc1 + ia;
        q.s16[o + l * D] = (__bf16)cs;
        q.s32[o + l * D] = cs;
        q.c32[o + l * D] = cc1;
    }
}

// ---- ssm_red: p = mean x_embed + d + mean_l y_l silu(s_l), w = mean_l y_l silu'(s_l) c_l
__global__ __launch_bounds__(64 * kSsmChunks) void ssm_red_kernel(RegionArgs q, int64_t p0)
{
    __shared__ float r1[kSsmChunks][64], r2[kSsmChunks][64];
    const int64_t z = blockIdx.y, pr = p0 + z, k = pr / q.B, b = pr % q.B;
    const int cc = threadIdx.x & 63, ch = threadIdx.x >> 6;
    const int dch = blockIdx.x * 64 + cc;
    const int D = q.D;
    const int64_t L = q.L;
    const int64_t per = (L + kSsmChunks - 1) / kSsmChunks;
    const int64_t l0 = ch * per < L ? ch * per : L;
    const int64_t l1 = l0 + per < L ? l0 + per : L;
    const int64_t o = z * L * D + dch;
    float u1 = 0.0f, u2 = 0.0f;
#pragma unroll 8
    for (int64_t l = l0; l < l1; ++l) {
        const float y = q.y32[o + l * D], sv = q.s32[o + l * D];
        u1 = fmaf(y, silu(sv), u1);
        u2 = fmaf(y * dsilu(sv), q.c32[o + l * D], u2);
    }
    r1[ch][cc] = u1;
    r2[ch][cc] = u2;
    __syncthreads();
    if (ch == 0) {
        float t1 = 0.0f, t2 = 0.0f;
        for (int u = 0; u < kSsmChunks; ++u) {
            t1 += r1[u][cc];
            t2 += r2[u][cc];
        }
        const float inv = 1.0f / (float)L;
        const int64_t bk = b * q.K + k;
        q.p[bk * D + dch] = q.xbar[b * D + dch] + q.d[bk * D + dch] + t1 * inv;
        q.wv[z * D + dch] = t2 * inv;
    }
}

// Workgroup order of the two big tangent products: workgroup i runs on XCD
// i % 8, so logical tile lg = (i % 8) (n / 8) + i / 8 gives each XCD a
// contiguous range of logical tiles, which then share an operand in that
// XCD's L2.
__device__ __forceinline__ int64_t xcd_order(int64_t i, int64_t n)
{
    return n % 8 == 0 ? (i % 8) * (n / 8) + i / 8 : i;
}

// ---- the first tangent product: Vt[z] = (S W1[k]^T) * silu'(u)[l][x] with
//      S[l r + j][d] = c_l[d] Jdec^T[pair][j][d], stored first (ssm_s) so that
//      both operands stream straight into LDS (gen_dma below) -----------------------
struct GenArgs {
    const __bf16 *S;    // [G][L r][D]
    const __bf16 *W1;   // [K][X][D]
    const float *g32;   // [G][L][X]
    __bf16 *Vt;         // [G][L r][X]
    int64_t L, p0, Bn;
    int D, X, rs;
    int ntn, ntm;       // 256-wide column tiles, 256-row tiles of a pair
    int64_t ntiles;
};

// ---- the second tangent product: Tpart[z][c][j][d] = sum over the tokens l of
//      256-row tile c of silu(s_l)[d] (Vt[z] W2[k]^T)[l r + j][d] ------------------
struct TokArgs {
    const __bf16 *Vt;   // [G][L r][X]
    const __bf16 *W2;   // [K][D][X]
    const float *s32;   // [G][L][D]
    float *Tpart;       // [G][nchunk][r][D], nchunk = the 256-row tiles of L r
    int64_t L, p0, Bn;  // pair z is p0 + z, of region (p0 + z) / Bn
    int X, D, r, rs, nchunk;
    int64_t ntiles;
};

// ---- ssm_s: the first tangent product's left operand S (GenArgs above), rounded
//      to bf16 as it is formed; thread e writes the 8 values of chunk e % (D / 8)
//      of row e / (D / 8) --------------------------------------------------------------
__global__ __launch_bounds__(kT) void ssm_s_kernel(RegionArgs q, int64_t p0)
{
    const int64_t z = blockIdx.y;
    const int D = q.D, r = q.r, dq = D / 8;
    const int64_t Lr = q.L * r;
    const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= Lr * dq)
        return;
    const int64_t row = e / dq, l = row / r;
    const int c = (int)(e % dq), j = (int)(row % r);
    const float *cp = q.c32 + (z * q.L + l) * D + c * 8;
    const f4 c0 = *(const f4 *)cp, c1 = *(const f4 *)(cp + 4);
    const bf16x8 jv = *(const bf16x8 *)(q.JdT + ((p0 + z) * r + j) * D + c * 8);
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[i] = (__bf16)(c0[i] * (float)jv[i]);
        o[4 + i] = (__bf16)(c1[i] * (float)jv[4 + i]);
    }
    *(bf16x8 *)(q.S16 + (z * Lr + row) * D + c * 8) = o;
}

// ==== 256 x 256 tiles with operands loaded straight into LDS ===========================
// C (256 x 256, fp32 in registers) = A rows x B rows^T over K, both bf16 with K
// contiguous.  Eight waves (2 x 4) of 128 x 64.  Two LDS stages of 64 k
// (32 KB per operand): the next stage's loads run while this stage's MFMAs
// do, one barrier per stage.  buffer_load_dwordx4 ... lds writes each lane's
// 16 bytes at M0 + 16 lane, so the operands take no registers and no VALU or
// LDS-write instructions; the rows (128 B) sit two to a 256-byte line with
// chunk q of row R in slot ((R & 1) 8 + q) ^ ((R / 2) & 7), the layout of
// lds_off, and each lane loads the global chunk that its LDS slot holds.
//
// A workgroup per CU takes one tile after another, and a tile's first stage
// loads beside the last products of the tile before it: with a workgroup per
// tile, its start, the latency of that first stage and of the weights, and the
// end of its stores came on top of every tile.  The weights of a tile (the rows
// of a [tokens][columns] fp32 array, 16 KB at most) load into LDS beside the
// second stage.  2 sequences x 4 regions, L 1024, D 768, X 1536, r 64: gen_dma
// 1448 -> 1391 us, tok_dma 1250 -> 1140, the call 3074 -> 2890.  The
// matrix cores are 44% and 56% busy, and 64 KB per stage and CU come from L2 at 7.1
// and 8.0-8.7 TB/s, which is not its limit (region_dma reads 13.8): a stage takes
// 2.0-2.4 us with one in flight.  Reading half a stage ahead of the products, other
// row pitches of S and Vt, and four stages of half the depth did not help.
constexpr int kDT = 512;                  // threads
constexpr int kDOp = 256 * BK * 2;        // bytes of one operand's stage (32 KB)
constexpr int kDStage = 2 * kDOp;         // A and B
constexpr int kDLoads = kDOp / 1024 / 8;  // 1 KB loads per wave, operand and stage
constexpr int kDWeights = 16 * 256 * 4;   // weights of a tile: at most 16 tokens
constexpr int kDLds = 2 * kDStage + kDWeights;

// A tile: resources of its operands' rows (ending at the last valid row, so no
// load leaves them; the epilogues do not rely on what the products of rows past
// it hold) and of its weights (from the tile's first token and column, rows ldw
// bytes apart).
struct DTile {
    i4 rsA, rsB, rsW;
};

// x, as a value that the compiler does not know to be the same in every tile: an
// epilogue's addresses, worked out before the loop and kept, do not fit the
// registers beside the product.
__device__ __forceinline__ int fresh(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The tiles i = blockIdx.x, + gridDim.x, ... below n: setup(i) gives the tile,
// epilogue(i, acc) weights and stores it.
template <typename Setup, typename Epi>
__device__ __forceinline__ void dtile_loop(int64_t n, int K, int tokens, int ldw, int w, int lane,
                                           uint32_t lbase, Setup &&setup, Epi &&epilogue)
{
    typedef __attribute__((address_space(3))) char lchar;
    const int wm = w >> 2, wn = w & 3;
    // load d of a wave (1 KB, rows 8 d' .. 8 d' + 7 with d' = w + 8 d): lane ->
    // line rp = 4 d' + lane / 16, row 2 rp + (lane & 15) / 8, global chunk
    // (lane & 7) ^ (rp & 7)
    int vo[kDLoads];
#pragma unroll
    for (int d = 0; d < kDLoads; ++d) {
        const int rp = 4 * (w + 8 * d) + (lane >> 4);
        vo[d] = (2 * rp + ((lane & 15) >> 3)) * K * 2 + (((lane & 7) ^ (rp & 7)) << 4);
    }
    // stage s of a tile into buffer buf
    auto issue = [&](const DTile &t, int s, int buf) {
        const uint32_t st = lbase + (uint32_t)(buf * kDStage);
#pragma unroll
        for (int d = 0; d < kDLoads; ++d) {
            const uint32_t blk = (uint32_t)((w + 8 * d) * 1024);
            dma_b128(__builtin_amdgcn_readfirstlane(st + blk), t.rsA, vo[d], s * BK * 2);
            dma_b128(__builtin_amdgcn_readfirstlane(st + kDOp + blk), t.rsB, vo[d], s * BK * 2);
        }
    };
    // operand reads: row lane & 15 of a 16-row block, chunk 4 ks + lane / 16
    uint32_t ro[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        ro[ks] = (uint32_t)(lds_off(lane & 15, 4 * ks + (lane >> 4)) * 2);
    const int nk = K / BK;
    int64_t i = blockIdx.x;
    if (i >= n)
        return;
    DTile cur = setup(i);
    issue(cur, 0, 0);
    int buf = 0;  // of the tile's next stage
    bool landed = false;  // this wave's share of it has arrived
    for (;;) {
        const int64_t inext = i + gridDim.x;
        f4 acc[8][4];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[a][b] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        DTile next = cur;
        for (int t = 0; t < nk; ++t) {
            // stage t complete; stage t - 1 (or the last tile's) read by every wave
            if (t == 0 && landed)
                lds_barrier();
            else
                dma_barrier<0>();
            if (t == 0)
                for (int l = w; l < tokens; l += 8)
                    dma_b128(__builtin_amdgcn_readfirstlane(
                                 lbase + (uint32_t)(2 * kDStage + l * 1024)),
                             cur.rsW, l * ldw + lane * 16, 0);
            if (t + 1 < nk) {
                issue(cur, t + 1, buf ^ 1);
            } else if (inext < n) {
                next = setup(inext);
                issue(next, 0, buf ^ 1);
            }
            const uint32_t st = lbase + (uint32_t)(buf * kDStage);
            buf ^= 1;
            bf16x8 a[2][8], b[2][4];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    a[ks][e] = *(const bf16x8 *)(lchar *)(uintptr_t)(st + ro[ks] +
                                                                      (wm * 128 + e * 16) * 128);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    b[ks][e] = *(const bf16x8 *)(lchar *)(uintptr_t)(st + kDOp + ro[ks] +
                                                                      (wn * 64 + e * 16) * 128);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int f = 0; f < 4; ++f)
                        acc[e][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][e], b[ks][f],
                                                                             acc[e][f], 0, 0, 0);
            // all operand reads first, then the MFMAs (each waits only for its own)
            __builtin_amdgcn_sched_group_barrier(0x100, 24, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 64, 0);
        }
        // The next tile's first stage (and, with one stage, the weights) before the
        // epilogue's own memory operations: it was issued a stage of products ago, and
        // a wait behind the stores would have to know how many the compiler made.
        if (nk == 1)
            dma_barrier<0>();
        else
            dma_wait();
        landed = true;
        epilogue(i, acc);
        if (inext >= n)
            return;
        cur = next;
        i = inext;
    }
}

// ---- gen_dma: the first tangent product (GenArgs above); the epilogue scales a
//      tile by silu'(u) and stores it in bf16 -------------------------------------
__global__ __launch_bounds__(kDT) __attribute__((amdgpu_waves_per_eu(2, 2))) void gen_dma_kernel(
    GenArgs a)
{
    __shared__ __attribute__((aligned(1024))) char smem[kDLds];
    typedef __attribute__((address_space(3))) char lchar;
    const uint32_t lbase = (uint32_t)(uintptr_t)(lchar *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t Lr = a.L << a.rs;
    const int D = a.D;
    struct At {
        int64_t z, row0, col0;
    };
    auto at = [&](int64_t i) {
        const int64_t lg = xcd_order(i, a.ntiles);
        return At{lg / ((int64_t)a.ntn * a.ntm), (lg / a.ntn) % a.ntm * 256, lg % a.ntn * 256};
    };
    auto setup = [&](int64_t i) {
        const At t = at(i);
        const int64_t k = (a.p0 + t.z) / a.Bn, l0 = t.row0 >> a.rs;
        const int vA = Lr - t.row0 < 256 ? (int)(Lr - t.row0) : 256;
        const int vB = a.X - t.col0 < 256 ? (int)(a.X - t.col0) : 256;
        return DTile{dma_rsrc(a.S + (t.z * Lr + t.row0) * D, (uint32_t)vA * D * 2),
                     dma_rsrc(a.W1 + (k * a.X + t.col0) * D, (uint32_t)vB * D * 2),
                     dma_rsrc(a.g32 + (t.z * a.L + l0) * a.X + t.col0,
                              (uint32_t)((((vA - 1) >> a.rs) * a.X + vB) * 4))};
    };
    // (a 16-row block is one token: r is a multiple of 16)
    const int wm = w >> 2, wn = w & 3;
    auto epilogue = [&](int64_t i, f4(&acc)[8][4]) {
        const At t = at(i);
        const int ln = fresh(lane), li = ln & 15, g = ln >> 4;
        // Lane (g, li) holds columns li of the four 16-column blocks; a transpose
        // among the lanes of a quad gives it four neighbouring columns of block
        // li & 3, so that a row's 64 columns are one 128-byte piece of a store
        // (2-byte stores of 32-byte pieces drained for 5 us of a 29 us tile).
        // Two rows go through it packed in one register.
        const bool odd = li & 1, upper = li & 2;
        auto swap = [](uint32_t &x, uint32_t &y, bool up, auto mask) {
            const uint32_t got = fbits(xchg<decltype(mask)::value>(bitsf(up ? x : y)));
            x = up ? got : x;
            y = up ? y : got;
        };
        __bf16 *out = a.Vt + t.z * Lr * a.X;
        const int col = wn * 64 + (li & 3) * 16 + (li >> 2) * 4;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int rl = wm * 128 + e * 16;
            const int64_t rb = t.row0 + rl;
            if (rb >= Lr)
                break;
            float gs[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                gs[j] = *(const float *)(lchar *)(uintptr_t)(
                    lbase + (uint32_t)(2 * kDStage +
                                       ((rl >> a.rs) * 256 + wn * 64 + j * 16 + li) * 4));
#pragma unroll
            for (int v = 0; v < 4; v += 2) {
                uint32_t x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    x[j] = __builtin_bit_cast(
                        uint32_t, __builtin_convertvector(f2{acc[e][j][v] * gs[j],
                                                             acc[e][j][v + 1] * gs[j]}, bf16x2));
                swap(x[0], x[1], odd, std::integral_constant<int, 1>{});
                swap(x[2], x[3], odd, std::integral_constant<int, 1>{});
                swap(x[0], x[2], upper, std::integral_constant<int, 2>{});
                swap(x[1], x[3], upper, std::integral_constant<int, 2>{});
                if (t.col0 + col < a.X) {
                    __bf16 *o = out + (rb + 4 * g + v) * a.X + t.col0 + col;
                    *(u2 *)o = u2{(x[0] & 0xFFFFu) | x[1] << 16, (x[2] & 0xFFFFu) | x[3] << 16};
                    *(u2 *)(o + a.X) = u2{x[0] >> 16 | (x[1] & kHighHalf),
                                          x[2] >> 16 | (x[3] & kHighHalf)};
                }
            }
        }
    };
    dtile_loop(a.ntiles, D, 256 >> a.rs, a.X * 4, w, lane, lbase, setup, epilogue);
}

// ---- tok_dma: the second tangent product (TokArgs above) -------------------------
// A tile is one column tile of D and one 256-row tile c of a pair (a tile
// row's token is row / r, its j is row mod r); its partial sum goes to
// Tpart[z][c].  The product is weighted by silu(s_l) and summed over the
// tile's tokens: first over a wave's row blocks that share j (blocks i and
// i + NB, NB = min(r, 128) / 16), then across the tile's two row halves
// through LDS, in the stage that the next tile does not load into.
template <int RS>
__global__ __launch_bounds__(kDT) __attribute__((amdgpu_waves_per_eu(2, 2))) void tok_dma_kernel(
    TokArgs a)
{
    constexpr int NB = (RS >= 7 ? 128 : (1 << RS)) / 16;
    constexpr int NR = NB < 4 ? NB : 4;  // row blocks exchanged at a time (64 KB)
    __shared__ __attribute__((aligned(1024))) char smem[kDLds];
    typedef __attribute__((address_space(3))) char lchar;
    const uint32_t lbase = (uint32_t)(uintptr_t)(lchar *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 2, wn = w & 3;
    const int64_t nct = (a.D + 255) / 256;
    const int64_t Lr = a.L << RS;
    struct At {
        int64_t z, row0, col0;
        int c;
    };
    auto at = [&](int64_t i) {
        const int64_t lg = xcd_order(i, a.ntiles);
        const int c = (int)((lg / nct) % a.nchunk);
        return At{lg / (nct * a.nchunk), (int64_t)c * 256, lg % nct * 256, c};
    };
    auto setup = [&](int64_t i) {
        const At t = at(i);
        const int64_t k = (a.p0 + t.z) / a.Bn, l0 = t.row0 >> RS;
        const int vA = Lr - t.row0 < 256 ? (int)(Lr - t.row0) : 256;
        const int vB = a.D - t.col0 < 256 ? (int)(a.D - t.col0) : 256;
        return DTile{dma_rsrc(a.Vt + (t.z * Lr + t.row0) * a.X, (uint32_t)vA * a.X * 2),
                     dma_rsrc(a.W2 + (k * a.D + t.col0) * a.X, (uint32_t)vB * a.X * 2),
                     dma_rsrc(a.s32 + (t.z * a.L + l0) * a.D + t.col0,
                              (uint32_t)((((vA - 1) >> RS) * a.D + vB) * 4))};
    };
    const int nk = a.X / BK;
    int done = 0;  // tiles finished: the last stage of tile t was in buffer (t + 1) nk - 1 mod 2
    auto epilogue = [&](int64_t i, f4(&acc)[8][4]) {
        const At t = at(i);
        const int ln = fresh(lane), li = ln & 15, g = ln >> 4;
        // (rows past L r are left out by selects: their products may be anything)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int rl = wm * 128 + e * 16;
            const bool live = t.row0 + rl < Lr;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float wt = silu(*(const float *)(lchar *)(uintptr_t)(
                    lbase + (uint32_t)(2 * kDStage +
                                       ((rl >> RS) * 256 + wn * 64 + j * 16 + li) * 4)));
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float x = live ? wt * acc[e][j][v] : 0.0f;
                    if (e < NB)
                        acc[e][j][v] = x;
                    else
                        acc[e % NB][j][v] += x;
                }
            }
        }
        // the lower row half adds the upper one's sums through LDS ([j][256] fp32)
        const uint32_t red = lbase + (uint32_t)((((done + 1) * nk - 1) & 1) * kDStage);
        ++done;
        float *out = a.Tpart + (t.z * a.nchunk + t.c) * ((int64_t)a.D << RS);
#pragma unroll
        for (int h = 0; h < NB; h += NR) {
            __syncthreads();  // (the operand reads, or the sums before, are done)
            if (wm == 1) {
#pragma unroll
                for (int e = 0; e < NR; ++e)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            *(float *)(lchar *)(uintptr_t)(
                                red + (uint32_t)(((e * 16 + 4 * g + v) * 256 + wn * 64 +
                                                  j * 16 + li) * 4)) = acc[h + e][j][v];
            }
            __syncthreads();
            if (wm == 0) {
#pragma unroll
                for (int e = 0; e < NR; ++e)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int cl = wn * 64 + j * 16 + li;
                        if (t.col0 + cl < a.D) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int jr = e * 16 + 4 * g + v;
                                out[(int64_t)(h * 16 + jr) * a.D + t.col0 + cl] =
                                    acc[h + e][j][v] +
                                    *(const float *)(lchar *)(uintptr_t)(
                                        red + (uint32_t)((jr * 256 + cl) * 4));
                            }
                        }
                    }
            }
        }
    };
    dtile_loop(a.ntiles, a.X, 256 >> RS, a.D * 4, w, lane, lbase, setup, epilogue);
}

// ---- tfin: dp^T[pair][j][d] = Jdec^T (1 + w[d]) + (1/L) sum_c Tpart[z][c][j][d] ----
__global__ __launch_bounds__(kT) void tfin_kernel(RegionArgs q, int64_t p0)
{
    const int64_t z = blockIdx.y, pr = p0 + z;
    const int D = q.D, r = q.r;
    const int idx = blockIdx.x * kT + threadIdx.x;
    if (idx >= r * D)
        return;
    const int j = idx / D, dch = idx % D;
    // four running sums over the row tiles' partials, so that four loads are
    // in flight at a time
    const float *tp = q.Tpart + (z * q.nchunk * r + j) * (int64_t)D + dch;
    const int64_t stride = (int64_t)r * D;
    float t4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int c = 0;
    for (; c + 4 <= q.nchunk; c += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            t4[u] += tp[(c + u) * stride];
    }
    for (; c < q.nchunk; ++c)
        t4[0] += tp[c * stride];
    const float t = (t4[0] + t4[1]) + (t4[2] + t4[3]);
    const int64_t o = (pr * r + j) * D + dch;
    q.dpT[o] = (__bf16)((float)q.JdT[o] * (1.0f + q.wv[z * D + dch]) + t / (float)q.L);
}

// Rows of a product's tiles: 128 while such tiles give every CU two, else 64,
// and 32 where 64-row tiles do not give every CU one.  At M = 128, N = K = 768
// over 8 regions 128-wide tiles are 48 workgroups of 12 serial steps (19.5 us),
// 32-row ones 384 (18 us with the bmv of 3072 rows beside it); the whole
// token-wise call of 2 sequences, 8 regions, 2048 tokens 442 -> 273 us with
// the joined launches and the token parts, 3 x 5 x 333 tokens (D 320, r 32)
// 172 -> 65, 1 x 1 x 17 93 -> 41, 8 x 16 x 2048 1660 -> 1566.
int gemm_tile(const GemmOp &g, int64_t batch)
{
    return gemm_blocks(g, batch, 128) >= 512 ? 128 : gemm_blocks(g, batch, 64) > 256 ? 64 : 32;
}
// Sequences per wave of a bmv: 2 where there are no more.
int bmv_nb(int64_t B) { return B <= 2 ? 2 : 8; }

// f(integral_constant) for a runtime choice of tile rows
template <typename F> void with_tile(int tm, F &&f)
{
    if (tm == 128)
        f(std::integral_constant<int, 128>{});
    else if (tm == 64)
        f(std::integral_constant<int, 64>{});
    else
        f(std::integral_constant<int, 32>{});
}

hipError_t gemm(const GemmOp &g, int64_t batch, hipStream_t st)
{
    const int tm = gemm_tile(g, batch);
    const dim3 grid = list_grid(gemm_blocks(g, batch, tm));
    with_tile(tm, [&](auto tag) {
        hipLaunchKernelGGL(gemm_nt_kernel<decltype(tag)::value>, grid, dim3(kT), 0, st, g, batch);
    });
    return hipGetLastError();
}

// a product over the K regions beside a bmv
hipError_t gemm_bmv(const GemmOp &g, const BmvArgs &v, int64_t K, hipStream_t st)
{
    const int tm = gemm_tile(g, K), nb = bmv_nb(v.B);
    const int64_t nv = round8(bmv_blocks(v.N, K, v.B, nb));
    const dim3 grid = list_grid(nv + gemm_blocks(g, K, tm));
    with_tile(tm, [&](auto tag) {
        constexpr int TM = decltype(tag)::value;
        if (nb == 2)
            hipLaunchKernelGGL((gemm_bmv_kernel<2, TM>), grid, dim3(kT), 0, st, g, v, nv, K);
        else
            hipLaunchKernelGGL((gemm_bmv_kernel<8, TM>), grid, dim3(kT), 0, st, g, v, nv, K);
    });
    return hipGetLastError();
}

hipError_t bmv(const BmvArgs &a, int64_t K, hipStream_t st)
{
    GemmOp none{};
    none.M = none.N = 0;  // no tiles
    return gemm_bmv(none, a, K, st);
}

// a product over the K regions beside the forward's LayerNorm
hipError_t gemm_ln(const GemmOp &g, const RegionArgs &q, hipStream_t st)
{
    const int tm = gemm_tile(g, q.K);
    const int64_t ng = gemm_blocks(g, q.K, tm);
    const dim3 grid = list_grid(ng + (q.B * q.K + 3) / 4);
    with_tile(tm, [&](auto tag) {
        hipLaunchKernelGGL(gemm_ln_kernel<decltype(tag)::value>, grid, dim3(kT), 0, st, g, ng, q);
    });
    return hipGetLastError();
}

// Dec_k and its operands, for both blocks: a = W_d1 m + b_d1 -> silu(a),
// silu'(a) beside the partial means of x_embed; then d = W_d2 silu(a) + b_d2,
// P1 and the means.
hipError_t dec(const RegionArgs &q, hipStream_t st)
{
    const int64_t K = q.K;
    const int D = q.D, r = q.r, nb = bmv_nb(q.B);
    const int64_t nch = (q.L + 63) / 64;
    BmvArgs v{(const __bf16 *)q.W_d1, (int64_t)D * r, q.m, K * r, r, q.b_d1, D, nullptr, 0, 0,
              nullptr, 0, 0, nullptr, q.su, q.sa, K * D, D, q.B, D, r};
    int64_t n0 = bmv_blocks(D, K, q.B, nb);
    dim3 grid = list_grid(n0 + nch * q.B);
    if (nb == 2)
        hipLaunchKernelGGL(in_kernel<2>, grid, dim3(kT), 0, st, q, v, n0);
    else
        hipLaunchKernelGGL(in_kernel<8>, grid, dim3(kT), 0, st, q, v, n0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    v = BmvArgs{(const __bf16 *)q.W_d2, (int64_t)D * D, q.su, K * D, D, q.b_d2, D, nullptr, 0, 0,
                nullptr, 0, 0, q.d, nullptr, nullptr, K * D, D, q.B, D, D};
    const int64_t np = q.B * K * (D / 64);
    grid = list_grid(n0 + np + q.B * ((D + kT - 1) / kT));
    if (nb == 2)
        hipLaunchKernelGGL(dec_kernel<2>, grid, dim3(kT), 0, st, q, v, n0, np);
    else
        hipLaunchKernelGGL(dec_kernel<8>, grid, dim3(kT), 0, st, q, v, n0, np);
    return hipGetLastError();
}

// The end of both blocks, from p, dp^T and silu(e), silu'(e): Enc_k beside T',
// the LayerNorm beside Jenc, and the Jacobian.
hipError_t enc(const RegionArgs &q, int rs, hipStream_t st)
{
    const int64_t K = q.K, Br = q.B * (int64_t)q.r;
    const int D = q.D, r = q.r;
    hipError_t e;
    // T'^T[k] = (dp^T W_e1[k]^T) * silu'(e)[b][k][h]    (B r x D, K = D)
    GemmOp g{q.dpT, D, Br * D, (const __bf16 *)q.W_e1, D, (int64_t)D * D, q.TT, D, Br * D, Br, D,
             D, q.se, D, K * (int64_t)D, rs, nullptr, true};
    // Enc = W_e2 silu(e) + b_e2
    const BmvArgs v{(const __bf16 *)q.W_e2, (int64_t)r * D, q.sue, K * D, D, q.b_e2, r, nullptr, 0,
                    0, nullptr, 0, 0, q.encv, nullptr, nullptr, K * r, r, q.B, r, D};
    if ((e = gemm_bmv(g, v, K, st)) != hipSuccess)
        return e;
    // Jenc^T[k] = T'^T W_e2[k]^T                        (B r x r, K = D), fp32
    g = GemmOp{q.TT, D, Br * D, (const __bf16 *)q.W_e2, D, (int64_t)r * D, q.JencT, r, Br * r, Br,
               r, D, nullptr, 0, 0, 0, nullptr, false};
    if ((e = gemm_ln(g, q, st)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(ln_jac_kernel, dim3((unsigned)(q.B * K)), dim3(kT),
                       (size_t)3 * r * sizeof(float), st, q);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_region_jacobians(const RegionArgs &q, hipStream_t st)
{
    const int64_t Br = q.B * (int64_t)q.r;
    const int D = q.D, X = q.X, r = q.r;
    const int64_t K = q.K;
    const __bf16 *Wd2 = (const __bf16 *)q.W_d2, *W1 = (const __bf16 *)q.W1;
    const __bf16 *W2 = (const __bf16 *)q.W2;
    // the interface width is a power of two (16 .. 128): scale rows by shift
    const int rs = r == 16 ? 4 : (r == 32 ? 5 : (r == 64 ? 6 : 7));
    hipError_t e;
    if ((e = dec(q, st)) != hipSuccess)
        return e;
    // Jdec^T[k] = P1[k] W_d2[k]^T                      (B r x D, K = D)
    GemmOp g{q.P1, D, Br * D, Wd2, D, (int64_t)D * D, q.JdT, D, Br * D, Br, D, D,
             nullptr, 0, 0, 0, nullptr, true};
    // cvec = W1 d
    BmvArgs v{W1, (int64_t)X * D, q.d, K * D, D, nullptr, 0, nullptr, 0, 0, nullptr, 0, 0, q.cvec,
              nullptr, nullptr, K * X, X, q.B, X, D};
    if ((e = gemm_bmv(g, v, K, st)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(region_dma_kernel, list_grid(K * q.B * (X / BN) * q.nsplit), dim3(kT), 0, st,
                       q);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    // U'^T[k] = (Jdec^T W1[k]^T) * gbar[b][k][x]        (B r x X, K = D)
    const int64_t part = q.B * K * X;  // sbar, gbar: nsplit partial means
    g = GemmOp{q.JdT, D, Br * D, W1, D, (int64_t)X * D, q.UT, X, Br * X, Br, X, D,
               q.gbar, X, K * (int64_t)X, rs, nullptr, true};
    g.nscale = q.nsplit;
    g.scale_ss = part;
    // p = W2 sbar + d + mean_l x_embed
    v = BmvArgs{W2, (int64_t)D * X, q.sbar, K * X, X, nullptr, 0, q.d, K * D, D,
                q.xbar, D, 0, q.p, nullptr, nullptr, K * D, D, q.B, D, X, q.nsplit, part};
    if ((e = gemm_bmv(g, v, K, st)) != hipSuccess)
        return e;
    // dp^T[k] = U'^T W2[k]^T + Jdec^T                   (B r x D, K = X)
    g = GemmOp{q.UT, X, Br * X, W2, X, (int64_t)D * X, q.dpT, D, Br * D, Br, D, X,
               nullptr, 0, 0, 0, q.JdT, true};
    // e = W_e1 p + b_e1 -> silu(e) (sue), silu'(e) (se)
    v = BmvArgs{(const __bf16 *)q.W_e1, (int64_t)D * D, q.p, K * D, D, q.b_e1, D, nullptr, 0, 0,
                nullptr, 0, 0, nullptr, q.sue, q.se, K * D, D, q.B, D, D};
    if ((e = gemm_bmv(g, v, K, st)) != hipSuccess)
        return e;
    return enc(q, rs, st);
}

}  // namespace lbi

namespace lbi {

hipError_t launch_region_jacobians_ssm(const RegionArgs &q, hipStream_t st)
{
    const int64_t BKn = q.B * q.K;
    const int64_t Br = q.B * (int64_t)q.r;
    const int D = q.D, X = q.X, r = q.r;
    const int64_t K = q.K, L = q.L;
    const int rs = r == 16 ? 4 : (r == 32 ? 5 : (r == 64 ? 6 : 7));
    const __bf16 *Wd2 = (const __bf16 *)q.W_d2, *W1 = (const __bf16 *)q.W1;
    const __bf16 *W2 = (const __bf16 *)q.W2;
    hipError_t e;
    if ((e = dec(q, st)) != hipSuccess)
        return e;
    GemmOp g;
    // Jdec^T[k] = P1[k] W_d2[k]^T                      (B r x D, K = D)
    g = GemmOp{q.P1, D, Br * D, Wd2, D, (int64_t)D * D, q.JdT, D, Br * D, Br, D, D,
               nullptr, 0, 0, 0, nullptr, true};
    if ((e = gemm(g, q.K, st)) != hipSuccess)
        return e;

    // the token-mixing block, G (sequence, region) pairs at a time
    const int64_t Lr = L * r;
    const int nctw = (D + 255) / 256;
    for (int64_t p0 = 0; p0 < BKn; p0 += q.G) {
        const int64_t gz = q.G < BKn - p0 ? q.G : BKn - p0;
        hipLaunchKernelGGL(ssm_fwd_kernel, dim3((unsigned)(D / 64), (unsigned)gz),
                           dim3(64 * kSsmChunks), 0, st, q, p0);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        // silu(u), silu'(u) for u = s W1[k]^T              (L x X, K = D)
        g = GemmOp{q.s16, D, L * D, W1, D, (int64_t)X * D, q.h16, X, L * X, L, X, D,
                   nullptr, 0, 0, 0, nullptr, true, p0, q.B, true, q.g32};
        if ((e = gemm(g, gz, st)) != hipSuccess)
            return e;
        // y = silu(u) W2[k]^T                               (L x D, K = X), fp32
        g = GemmOp{q.h16, X, L * X, W2, X, (int64_t)D * X, q.y32, D, L * D, L, D, X,
                   nullptr, 0, 0, 0, nullptr, false, p0, q.B, false, nullptr};
        if ((e = gemm(g, gz, st)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(ssm_red_kernel, dim3((unsigned)(D / 64), (unsigned)gz),
                           dim3(64 * kSsmChunks), 0, st, q, p0);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        // S = c_l Jdec^T (bf16), then Vt = (S W1[k]^T) * silu'(u)[l][x]   (L r x X, K = D)
        hipLaunchKernelGGL(ssm_s_kernel, dim3((unsigned)((Lr * (D / 8) + kT - 1) / kT),
                                              (unsigned)gz),
                           dim3(kT), 0, st, q, p0);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        const int ntn = (X + 255) / 256, ntm = (int)((Lr + 255) / 256);
        const int64_t gtiles = (int64_t)ntn * ntm * gz;
        GenArgs ga{q.S16, W1, q.g32, q.Vt, L, p0, q.B, D, X, rs, ntn, ntm, gtiles};
        hipLaunchKernelGGL(gen_dma_kernel, dim3((unsigned)(gtiles < kCUs ? gtiles : kCUs)),
                           dim3(kDT), 0, st, ga);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        const int64_t ttiles = (int64_t)nctw * q.nchunk * gz;
        TokArgs ta{q.Vt, W2, q.s32, q.Tpart, L, p0, q.B, X, D, r, rs, q.nchunk, ttiles};
        const dim3 tgrid((unsigned)(ttiles < kCUs ? ttiles : kCUs));
        if (rs == 4)
            hipLaunchKernelGGL(tok_dma_kernel<4>, tgrid, dim3(kDT), 0, st, ta);
        else if (rs == 5)
            hipLaunchKernelGGL(tok_dma_kernel<5>, tgrid, dim3(kDT), 0, st, ta);
        else if (rs == 6)
            hipLaunchKernelGGL(tok_dma_kernel<6>, tgrid, dim3(kDT), 0, st, ta);
        else
            hipLaunchKernelGGL(tok_dma_kernel<7>, tgrid, dim3(kDT), 0, st, ta);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        hipLaunchKernelGGL(tfin_kernel, dim3((unsigned)((r * D + kT - 1) / kT), (unsigned)gz),
                           dim3(kT), 0, st, q, p0);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }

    // e = W_e1 p + b_e1 -> silu(e), silu'(e), and the end as for the token-wise
    // block
    const BmvArgs v{(const __bf16 *)q.W_e1, (int64_t)D * D, q.p, K * D, D, q.b_e1, D, nullptr, 0, 0,
                    nullptr, 0, 0, nullptr, q.sue, q.se, K * D, D, q.B, D, D};
    if ((e = bmv(v, K, st)) != hipSuccess)
        return e;
    return enc(q, rs, st);
}

}  // namespace lbi
