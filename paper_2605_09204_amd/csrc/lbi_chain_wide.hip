// The chain scan for fp32 storage at r = 128 in the split arithmetic: four
// matrix waves and four staging waves per chain segment, A_j in column panels.
//
// It computes what the workgroup chain kernel computes: the suffix composites
// P_j = A_j P_{j+1}, c_j = A_j c_{j+1} + b_j of a segment (Proposition "Scan
// Formulation of Backpropagation"), written out, or applied as they form,
// lambda_j = P_j lambda_K + c_j (Algorithm "Bounded-Interface Backpropagation",
// Phase 2).  The workgroup kernel has no split form at this width, because two
// tiles of three bf16 planes (192 KB) do not fit LDS; its fp32 matrix cores
// need 6.8 us for a slot's product, the six bf16 products 2.6.
//
//   * Panels.  A_j goes through LDS 32 columns at a time (the k range of one
//     MFMA): 128 x 32 values as three bf16 planes, 24 KB, two buffers, one
//     barrier per panel, four panels per slot.  A row's 32 values sit in
//     operand order in four 16-byte chunks, swizzled over 16 slots of a
//     256-byte line of four rows, so that operand reads and staging writes
//     touch all banks.
//   * Matrix waves (w < 4) hold column blocks w and w + 4 of P in the
//     accumulator layout, which is the B operand layout of the next product,
//     as in the workgroup kernel.  Per panel and wave: 24 operand reads, 96
//     MFMAs, and the split of the next panel's 16 P values per lane between
//     them; the apply of slot j+1 runs beside the second panel's products.
//     Eight waves of one column block each would read A twice as often, as
//     many LDS cycles as the MFMAs take; that is why only four form products.
//   * Staging waves, one beside each matrix wave on its SIMD, load A a slot
//     ahead (two slots with a widths hint; 16-byte buffer loads), split it, form c_j from the same registers
//     and store lambda.  Neither role's registers are live in the other's loop.
//
//   * Range.  Three bf16 parts hold an fp32 value to its last bit from 2^-110 up
//     to where it rounds to an infinity in bf16 (about 3.396e38); an infinity, or
//     a value past that, leaves NaN parts, and a smaller one keeps only its bits
//     from 2^-133 up.  A P that fades is therefore scaled by 2^64, once, long before
//     that: with lambda by each matrix wave for its columns, where a sum over them
//     falls below 2^-64 of lambda_K's largest entry there.  A segment in which a loss
//     can show all the same is done again from its end on the fp32 matrix cores
//     (exact_pass), so the results are those of float32 products.  What shows it,
//     with lambda: such a sum below 2^-96 before P is scaled, and a row of lambda_s
//     that is not finite, or not zero and below 2^-96 of itself at s + 1 (what was
//     lost is otherwise below 2^-29 of a row).  With composites, the largest magnitude
//     of a quarter column of P_s (a lane's): 2^126 or more, or not zero and below
//     2^-96 (until P is scaled) or below 2^-96 of the quarter's at s + 1; and a NaN in
//     the segment's last composite.  The checks cost up to 4% of a lambda pass without
//     affine terms, 1% of others, and 5% of a hinted composite pass.  A segment done
//     again takes 11-12 us a slot (scan_chain_kernel on the fp32 matrix cores 9).
//
// What bounds it: a slot is 384 MFMAs of 16 cycles per SIMD (2.6 us at the top
// clock), with about 500 VALU instructions of the matrix wave beside them; with
// every CU busy the MFMAs run at 1.0-1.2 PFLOP/s of bf16 products, where a
// large library matrix product reaches 1.4 on the same card.  192 chains of 24
// slots: 119 us against 218 with the workgroup kernel on the fp32 matrix cores;
// 256 x 128: 757 against 1163; widths cycling 32/64/128, 1024 x 64: 675 against
// 807 (compact storage 698 against 790).
//
// All HIP code here is built with packed fp32 math disabled.

#include <type_traits>

#include "lbi_device.hpp"
#include "lbi_internal.h"

namespace lbi {
namespace {

constexpr int kR = 128;
constexpr int kNP = 4;                       // panels per tile
constexpr int kPC = kR / kNP;                // panel columns
constexpr int kPlane = kR * kPC;             // elements of one plane of a panel
constexpr int kTileBytes = kR * kR * 4;

// Element offset of 16-byte chunk q (0..3) of panel row r.
__device__ __forceinline__ int panel_pos(int r, int q)
{
    const int line = r >> 2;
    return line * 128 + ((r & 3) * 4 + (q ^ (line & 3))) * 8;
}

// The range checks' bounds (see Range above).
constexpr float kShow = 0x1p-96f, kFull = 0x1p126f;
// Below kFade P is multiplied by kUp, once a segment, and what is formed from it by
// kDown: a P that fades then stays in the split's range (float32 itself ends before
// the scaled values leave it again).
constexpr float kFade = 0x1p-64f, kUp = 0x1p64f, kDown = 0x1p-64f;

// The three parts of a lane's B operand: 4 rows of two row blocks of P.
struct Parts {
    bf16x8 h, m, l;
};
__device__ __forceinline__ Parts split_rows(const f4 &a, const f4 &b)
{
    const Split2 s0 = split_pair_keep(a[0], a[1]), s1 = split_pair_keep(a[2], a[3]);
    const Split2 s2 = split_pair_keep(b[0], b[1]), s3 = split_pair_keep(b[2], b[3]);
    return {__builtin_bit_cast(bf16x8, u4{s0.h, s1.h, s2.h, s3.h}),
            __builtin_bit_cast(bf16x8, u4{s0.m, s1.m, s2.m, s3.m}),
            __builtin_bit_cast(bf16x8, u4{s0.l, s1.l, s2.l, s3.l})};
}

// The larger of m and the magnitudes in a column's rows of two row blocks.
__device__ __forceinline__ float column_top(float m, const f4 &a, const f4 &b)
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
        m = fmaxf(fmaxf(m, fabsf(a[v])), fabsf(b[v]));
    return m;
}

// Row v of a lane's blocks P[t], times lk.
template <int NT>
__device__ __forceinline__ float column_sum(const f4 (&P)[NT], int v, const float (&lk)[NT])
{
    if constexpr (NT == 1)
        return P[0][v] * lk[0];
    else
        return P[0][v] * lk[0] + P[1][v] * lk[1];
}

// acc += A panel x b for the first NR row blocks and NT column blocks of a wave;
// pan: this lane's operand of row block 0 (row block I adds 512 I elements).
// Row blocks go in groups that give four independent accumulators.
template <int NR, int NT, int W>
__device__ __forceinline__ void panel_product(f4 (&acc)[8][W], const __bf16 *pan,
                                              const Parts (&b)[W])
{
    constexpr int GI = NT == 1 && NR >= 4 ? 4 : 2;
#pragma unroll
    for (int I0 = 0; I0 < NR; I0 += GI) {
        bf16x8 ah[GI], am[GI], al[GI];
#pragma unroll
        for (int i = 0; i < GI; ++i) {
            ah[i] = *(const bf16x8 *)(pan + 512 * (I0 + i));
            am[i] = *(const bf16x8 *)(pan + kPlane + 512 * (I0 + i));
            al[i] = *(const bf16x8 *)(pan + 2 * kPlane + 512 * (I0 + i));
        }
#define LBI_WIDE_TERM(X, Y)                                                                   \
    _Pragma("unroll") for (int i = 0; i < GI; ++i)                                            \
        _Pragma("unroll") for (int t = 0; t < NT; ++t) acc[I0 + i][t] =                       \
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(X[i], b[t].Y, acc[I0 + i][t], 0, 0, 0);
        LBI_WIDE_TERM(ah, h)
        LBI_WIDE_TERM(ah, m)
        LBI_WIDE_TERM(am, h)
        LBI_WIDE_TERM(ah, l)
        LBI_WIDE_TERM(al, h)
        LBI_WIDE_TERM(am, m)
#undef LBI_WIDE_TERM
    }
}

// ---- a segment again, on the fp32 matrix cores (see Range above) ----------------
// One barrier per slot: the matrix waves hold P_s and form P_{s-1} = A_{s-1} P_s with
// their operands straight from global memory, the staging waves c_{s-1}; lambda is
// stored again from slot worst on, composites from the segment's end, and what is
// published counts on from npub publications.  c_s is in entry s & 1 of sC, the
// apply's sums of slot s in entry s & 1 of sPart.  The arguments and the thread's
// index are read anew, so that the loops before keep nothing for this in registers.
template <bool AFF, int HINT, int OUT, int NT>
__device__ __forceinline__ void exact_pass(int32_t worst, int64_t npub, float (*sC)[kR],
                                           float (*sPart)[4][kR])
{
    typedef const __attribute__((address_space(4))) ScanArgs *ArgsPtr;
    ArgsPtr pa = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(pa));
    const __attribute__((address_space(4))) ScanArgs &args = *pa;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    constexpr bool compact = HINT == kHintCompact;
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, li = lane & 15, st = tid - 256;
    const int64_t beta = blockIdx.x / args.S;
    const int64_t s0 = (int64_t)(blockIdx.x % args.S) * args.L;
    const int64_t K = args.K - s0 < args.L ? args.K - s0 : args.L;
    const int64_t first = beta * args.K + s0;
    const int64_t cslot = args.agg_only ? (int64_t)blockIdx.x : first;
    const float *A = (const float *)args.A +
                     (compact ? beta * (int64_t)args.totalA : first * (int64_t)(kR * kR));
    const float *bv = (const float *)args.b +
                      (compact ? beta * (int64_t)args.totalR : first * (int64_t)kR);
    auto blocks = [&](int64_t s) {
        return !HINT ? 8
               : s < 0 ? 0
                       : (int)((args.wcode[(s0 + s) >> 3] >> (((s0 + s) & 7) * 4)) & 15u);
    };
    auto pitch = [](int wc) { return compact ? 16 * wc : kR; };
    const int wK = blocks(K);
    int32_t offA = args.totalA, offR = args.totalR;  // (compact storage)
    if (compact) {
        offA -= 16 * blocks(K - 1) * pitch(wK);
        offR -= 16 * blocks(K - 1);
    }
    f4 P[8][NT];
    float lk[NT] = {};
    if (w < 4) {
        const int nrow = 16 * blocks(K - 1), ld = pitch(wK);
        const float *T = A + (compact ? (int64_t)offA : (K - 1) * (int64_t)(kR * kR));
#pragma unroll
        for (int I = 0; I < 8; ++I)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * I + 4 * g + v, col = 16 * (w + 4 * t) + li;
                    P[I][t][v] = row < nrow && col < ld ? T[row * ld + col] : 0.0f;
                }
        if constexpr (OUT == kOutLambda) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int idx = 16 * (w + 4 * t) + li, rK = compact ? 16 * wK : kR;
                lk[t] = idx >= rK     ? 0.0f
                        : args.lamSeg ? args.lamSeg[(int64_t)blockIdx.x * kR + idx]
                                      : ((const float *)args.lamK)[beta * rK + idx];
            }
        }
    } else if (st < kR) {
        const int nrow = compact ? 16 * blocks(K - 1) : kR;
        const int64_t at = compact ? (int64_t)offR : (K - 1) * (int64_t)kR;
        sC[(K - 1) & 1][st] = AFF && st < nrow ? bv[at + st] : 0.0f;
    }
    int32_t left = args.pchunk;
    int64_t points = 0, pub = -1;  // publications up to this slot; the pending one
    auto publish = [&]() {
        if (pub >= 0 && st == 0 && points > npub) {
            __hip_atomic_fetch_max(&args.progress[beta], (uint32_t)pub, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            if (args.pub_clock)
                args.pub_clock[beta * args.npub + npub] = __builtin_amdgcn_s_memrealtime();
            ++npub;
        }
        pub = -1;
    };
#pragma unroll 1
    for (int64_t s = K - 1; s >= 0; --s) {
        // A_{s-1}: nr row and wc column blocks
        const int wc = blocks(s), nr = blocks(s - 1), ld = pitch(wc);
        if (w < 4) {
            if constexpr (OUT == kOutLambda) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float q[16];
#pragma unroll
                    for (int I = 0; I < 4; ++I)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            q[4 * I + v] = column_sum<NT>(P[4 * h + I], v, lk);
                    group_reduce<16, 16>(q, li);
                    sPart[s & 1][w][64 * h + 16 * (li >> 2) + 4 * g + (li & 3)] = q[0];
                }
            } else if (!args.agg_only || s == 0) {
                float *T = args.Pout + (cslot + s) * (int64_t)(kR * kR) + 16 * w + li;
#pragma unroll
                for (int I = 0; I < 8; ++I)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            T[(16 * I + 4 * g + v) * kR + 64 * t] = P[I][t][v];
            }
        }
        __syncthreads();
        if (compact && s > 0)
            offA -= 16 * nr * ld;
        const float *T = A + (compact ? (int64_t)offA : (s - 1) * (int64_t)(kR * kR));
        if (w >= 4) {
            publish();
            const float c = sC[s & 1][st & (kR - 1)];
            if (OUT == kOutLambda && st < (compact ? 16 * wc : kR) && s <= worst)
                args.lam[(compact ? beta * (int64_t)args.totalR + offR
                                  : (first + s) * (int64_t)kR) + st] =
                    ((sPart[s & 1][0][st] + sPart[s & 1][1][st]) +
                     (sPart[s & 1][2][st] + sPart[s & 1][3][st])) +
                    c;
            if (OUT == kOutComposite && st < kR && args.cout && (!args.agg_only || s == 0))
                args.cout[(cslot + s) * kR + st] = c;
            if (OUT == kOutLambda && args.progress && (--left == 0 || s == 0)) {
                pub = K - s;
                ++points;
                left = args.pchunk;
                if (st < kR)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            }
            if (compact)
                offR -= 16 * nr;
            // two threads a row, half of its columns each
            const int row = st >> 1, nrow = compact ? 16 * nr : kR;
            const int ncol = (HINT ? 16 * wc : kR) / 2, col0 = (st & 1) * ncol;
            float x = 0.0f;
            if (AFF && s > 0 && row < nrow)
#pragma unroll 4
                for (int i = col0; i < col0 + ncol; i += 4) {
                    const f4 a = *(const f4 *)&T[row * ld + i], y = *(const f4 *)&sC[s & 1][i];
                    x += a[0] * y[0] + a[1] * y[1] + a[2] * y[2] + a[3] * y[3];
                }
            x += xchg<1>(x);
            if (AFF && s > 0 && row < nrow)
                x += bv[(compact ? (int64_t)offR : (s - 1) * (int64_t)kR) + row];
            if (s > 0 && (st & 1) == 0)
                sC[(s - 1) & 1][row] = x;
        } else if (s > 0) {
            // element v of row block k of P is the B operand of an MFMA over the rows
            // 16 k + 4 g + v; A's columns past wc blocks, and rows past nr, read as
            // zero (nothing of P is at those columns)
            const int voff = (li * ld + 4 * g) * 4;
            const uint64_t base = (uint64_t)(uintptr_t)T;
            void *const tile = (void *)(uintptr_t)(
                (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base) |
                (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32);
            auto load = [&](u4(&a)[8], int k) {
                const int bytes = !HINT ? kTileBytes : k < wc ? 16 * nr * ld * 4 : 0;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    tile, 0, __builtin_amdgcn_readfirstlane(bytes), kBufferWord3);
#pragma unroll
                for (int I = 0; I < 8; ++I)
                    a[I] = __builtin_amdgcn_raw_buffer_load_b128(
                        rs, voff, __builtin_amdgcn_readfirstlane((16 * I * ld + 16 * k) * 4), 0);
            };
            f4 Q[8][NT];
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    Q[I][t] = f4{0.0f, 0.0f, 0.0f, 0.0f};
            // (with a hint, only A_{s-1}'s column blocks and halves of its row blocks)
            u4 a[2][8];
            load(a[0], 0);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (HINT && k >= wc)
                    break;
                if (k < 7)
                    load(a[(k + 1) & 1], k + 1);
                // (here, a step of products ahead, and not later)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < 8; h += 4) {
                    if (HINT && h >= nr)
                        break;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int I = h; I < h + 4; ++I)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                Q[I][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    bitsf(a[k & 1][I][v]), P[k][t][v], Q[I][t], 0, 0, 0);
                }
            }
            // (with a hint, rows and columns that are not there stay zero: no zero
            // times an infinity)
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    P[I][t] = !HINT || (I < nr && w + 4 * t < wK) ? Q[I][t]
                                                                  : f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    if (OUT == kOutLambda && args.progress) {
        __syncthreads();
        if (w >= 4)
            publish();
    }
}

template <bool AFF, int HINT, int OUT, int NT>
__global__ __launch_bounds__(512) void scan_wide_kernel(const ScanArgs args)
{
    __shared__ __attribute__((aligned(16))) __bf16 sA[2][3 * kPlane];
    // c_s in entry s & 3; the apply's partial sums of slot s per matrix wave, in
    // entry s & 1
    __shared__ __attribute__((aligned(16))) float sC[4][kR];
    __shared__ __attribute__((aligned(16))) float sPart[OUT == kOutLambda ? 2 : 1][4][kR];
    // range: the latest slot whose results show a loss (-1: none).  Entry j & 1 holds
    // j when that was found in the loop's slot j; all waves read it in the next slot
    // and end the loop with that one (with a hint they go on to the last slot: another
    // way out of those loops costs them registers that they do not have)
    __shared__ int32_t sWorst, sFound[2];
    __shared__ int64_t sNpub;  // (streaming) publications made

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, li = lane & 15;
    // this workgroup's segment: slots s0 .. s0 + K - 1 of chain beta; below,
    // slot indices are local to the segment
    const int64_t beta = blockIdx.x / args.S;
    const int64_t s0 = (int64_t)(blockIdx.x % args.S) * args.L;
    const int64_t K = args.K - s0 < args.L ? args.K - s0 : args.L;
    const int64_t first = beta * args.K + s0;
    // (compact storage, whole chains: slot s's tile, b_s and lambda_s follow
    // those of slot s - 1 at their true sizes)
    constexpr bool compact = HINT == kHintCompact;
    const float *A = (const float *)args.A +
                     (compact ? beta * (int64_t)args.totalA : first * (int64_t)(kR * kR));
    const float *bv = AFF ? (const float *)args.b +
                                (compact ? beta * (int64_t)args.totalR : first * (int64_t)kR)
                          : nullptr;
    // composites at [B][K], or only the segment aggregates at [B][S]
    const int64_t cslot = args.agg_only ? (int64_t)blockIdx.x : first;
    // With a widths hint: 16-row blocks of slot s that can be nonzero (s = K:
    // the segment's end; 0 before the segment).  What the kernel leaves out
    // would add exact zeros.  A lookup is a scalar load, whose wait also drains
    // the LDS queue: the loops carry the codes they need and fetch one per slot,
    // a slot early.
    auto blocks = [&](int64_t s) {
        return !HINT ? 8 : s < 0 ? 0 : (int)((args.wcode[(s0 + s) >> 3] >> (((s0 + s) & 7) * 4)) & 15u);
    };
    // (writing composites, every row block is formed: the shapes of the product
    // do not fit the registers beside the stores)
    constexpr bool kShapes = HINT && OUT == kOutLambda;
    // panels of a tile with wc column blocks; its row pitch in storage
    auto panels = [](int wc) { return HINT ? (wc + 1) >> 1 : kNP; };
    auto pitch = [](int wc) { return compact ? 16 * wc : kR; };

    // entry idx of the segment end's lambda
    auto lambda_end = [&](int idx) {
        const int rK = compact ? 16 * blocks(K) : kR;
        return idx >= rK     ? 0.0f
               : args.lamSeg ? args.lamSeg[(int64_t)blockIdx.x * kR + idx]
                             : ((const float *)args.lamK)[beta * rK + idx];
    };
    if (tid < 2)
        sFound[tid] = -1;
    if (tid == 2)
        sWorst = -1;
    if (tid == 3)
        sNpub = 0;
    bool again = false;  // the slot loop ended early: the segment is done again

    if (w < 4) {
        // ---- matrix waves ---------------------------------------------------
        float lk[NT] = {};
        int up = 0;
        // (lambda) sums below fade show that P fades: it is then scaled, once
        float fade = 0.0f;
        bool fades = false;
        if constexpr (OUT == kOutLambda) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
                lk[t] = lambda_end(16 * (w + 4 * t) + li);
            // The wave's part of lambda_K is taken times 2^up, so that its largest entry
            // is at least 1 and no sum vanishes before the check below has seen it
            // (the sums are taken times 2^-up).
            float end = fabsf(lk[0]);
            if (NT == 2)
                end = fmaxf(end, fabsf(lk[NT - 1]));
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1)
                end = fmaxf(end, __shfl_xor(end, o));
            end = bitsf(__builtin_amdgcn_readfirstlane(fbits(end)));
            if (end > 0.0f && end < 1.0f) {
                up = 1 - __builtin_amdgcn_frexp_expf(end);
                end = 1.0f;
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    lk[t] = ldexpf(lk[t], up);
            }
            fade = end * kFade;
        }
        float *Pout = OUT == kOutComposite ? args.Pout + cslot * (int64_t)(kR * kR) : nullptr;
        bool faded = false;  // P is scaled, and what is formed from it is taken times down
        float down = 1.0f;
        // P_s, row blocks i0 .. i1 - 1, to global memory
        auto store_rows = [&](const f4(&P)[8][NT], int64_t s, int i0, int i1) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(Pout + s * (int64_t)(kR * kR)), 0, kTileBytes, kBufferWord3);
#pragma unroll
            for (int I = i0; I < i1; ++I)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        __builtin_amdgcn_raw_buffer_store_b32(
                            fbits(P[I][t][v] * down), rs,
                            ((16 * I + 4 * g + v) * kR + 16 * (w + 4 * t) + li) * 4, 0, 0);
        };
        // P_s lambda over this wave's columns, rows 64 h .. 64 h + 63
        auto apply = [&](const f4(&P)[8][NT], int64_t s, int h) {
            float q[16];
#pragma unroll
            for (int I = 0; I < 4; ++I)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    q[4 * I + v] = column_sum<NT>(P[4 * h + I], v, lk);
            group_reduce<16, 16>(q, li);
            // lane li holds value li (= 4 I + v)
            sPart[s & 1][w][64 * h + 16 * (li >> 2) + 4 * g + (li & 3)] = ldexpf(q[0], -up);
            const float a = fabsf(q[0]);
            const bool low = a > 0.0f && a < fade;
            if (__builtin_expect(__any(low), 0)) {
                fades = true;
                if (low && a < fade * (kShow * kUp)) {
                    atomicMax(&sWorst, (int32_t)s);
                    if (!HINT)
                        sFound[(s - 1) & 1] = (int32_t)(s - 1);
                }
            }
        };
        f4 P[8][NT];
        {
            const int nrow = 16 * blocks(K - 1), ld = pitch(blocks(K));
            const float *T = A + (compact ? (int64_t)args.totalA - nrow * ld
                                          : (K - 1) * (int64_t)(kR * kR));
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * I + 4 * g + v, col = 16 * (w + 4 * t) + li;
                        P[I][t][v] = row < nrow && col < ld ? T[row * ld + col] : 0.0f;
                    }
        }
        const int apos = panel_pos(li, g);  // row block I adds 512 I elements
        Parts b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
            b[t] = split_rows(P[0][t], P[1][t]);
        // (columns past the segment end's width are zero)
        const int nt = HINT && 4 + w >= blocks(K) ? 1 : 2;
        int buf = 0;  // the panel's LDS buffer
        // (composites) the largest magnitudes in this lane's rows of P's two columns, of
        // the row blocks split so far, and of a slot later
        float top[NT], before[NT], hard = kShow;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            top[t] = column_top(0.0f, P[0][t], P[1][t]);
            before[t] = 0.0f;
        }
        __syncthreads();
        auto scale_up = [&](f4(&X)[8][NT]) {
            faded = true;
            down = kDown;
            up += 64;
            fade = 0.0f;
            fades = false;
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    X[I][t] *= kUp;
        };
        // the range check of the P whose row blocks are all in top, in the loop's slot j
        // (-1: past it); true if it fades.  A NaN, which top leaves out, is in every row
        // of every composite after it: the last slot's check finds it.
        auto check_columns = [&](int64_t j, bool bad) {
            bool fades = false;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const float c = top[t];
                bad |= c >= kFull || (c > 0.0f && c < fmaxf(hard, before[t] * kShow));
                fades |= c > 0.0f && c < kFade;
                before[t] = c;
            }
            if (__builtin_expect(bad, 0)) {
                sWorst = 0;
                if (!HINT && j >= 0)
                    sFound[j & 1] = (int32_t)j;
            }
            if (faded)
                hard = 0.0f;
            return !faded && __any(fades);
        };
        // P_j (Pn) from P_{j+1} (P); b holds the split of P's first two row
        // blocks on entry, of Pn's on return
        int wr = blocks(K - 1), wnext = blocks(K - 2);
        // (true: the segment is to be done again)
        auto slot = [&](const f4(&P)[8][NT], f4(&Pn)[8][NT], int64_t j) {
            int32_t found = -1;
            const int wc = wr;
            [[maybe_unused]] const int np = panels(wc), nr = wnext;
            wr = wnext;
            wnext = blocks(j - 1);
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    Pn[I][t] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int p = 0; p < kNP; ++p) {
                if (HINT && p >= np)
                    break;
                __syncthreads();
                const __bf16 *pan = sA[HINT ? buf : p & 1] + apos;
                buf ^= 1;
                if (!HINT && p == 0)
                    found = sFound[(j + 1) & 1];
                Parts bn[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    bn[t] = b[t];
                if constexpr (kShapes) {
                    // (blocks past nr hold zeros)
                    auto rows_for = [&](auto ntag) {
                        constexpr int N = decltype(ntag)::value;
                        if (nr <= 2)
                            panel_product<2, N>(Pn, pan, b);
                        else if (nr <= 4)
                            panel_product<4, N>(Pn, pan, b);
                        else
                            panel_product<8, N>(Pn, pan, b);
                    };
                    if (NT == 1 || nt == 1)
                        rows_for(std::integral_constant<int, 1>{});
                    else
                        rows_for(std::integral_constant<int, NT>{});
                } else {
                    panel_product<8, NT>(Pn, pan, b);
                }
                if (p < kNP - 1) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        bn[t] = split_rows(P[2 * p + 2][t], P[2 * p + 3][t]);
                        if constexpr (OUT == kOutComposite)
                            top[t] = column_top(top[t], P[2 * p + 2][t], P[2 * p + 3][t]);
                    }
                }
                if constexpr (OUT == kOutLambda) {
                    // (a hinted slot may have one panel only)
                    if (HINT ? p == 0 : p == 1)
                        apply(P, j + 1, 0);
                    // (rows past wc blocks are zero, and finish() takes them so)
                    if (HINT ? p == 0 && wc > 4 : p == 2)
                        apply(P, j + 1, 1);
                } else if (!args.agg_only) {
                    if (!HINT)
                        store_rows(P, j + 1, 2 * p, 2 * p + 2);
                    else if (p == 0)
                        store_rows(P, j + 1, 0, 8);
                }
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    b[t] = bn[t];
            }
            if constexpr (OUT == kOutComposite) {
                if (__builtin_expect(check_columns(j, false), 0)) {
                    scale_up(Pn);
                    hard = kShow * kUp;  // of P_j, formed before it was scaled
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        before[t] *= kUp;
                }
            } else if (__builtin_expect(fades, 0)) {
                scale_up(Pn);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                b[t] = split_rows(Pn[0][t], Pn[1][t]);
                if constexpr (OUT == kOutComposite)
                    top[t] = column_top(0.0f, Pn[0][t], Pn[1][t]);
            }
            return !HINT && __builtin_amdgcn_readfirstlane(found) == (int32_t)(j + 1);
        };
        auto last = [&](const f4(&X)[8][NT]) {
            __syncthreads();
            if constexpr (OUT == kOutLambda) {
                apply(X, 0, 0);
                apply(X, 0, 1);
            } else {
                store_rows(X, 0, 0, 8);
                bool bad = false;
#pragma unroll
                for (int I = 0; I < 8; ++I)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        top[t] = column_top(top[t], X[I][t], X[I][t]);
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            bad |= X[I][t][v] != X[I][t][v];
                    }
                check_columns(-1, bad);
            }
        };
        // (the barrier: lambda_2's sums, in slot 0's entry, may still be read in
        // the last phase)
        f4 Q[8][NT];
        int64_t j = K - 2;
        if constexpr (HINT) {
            for (; j >= 0; --j) {
                slot(P, Q, j);
#pragma unroll
                for (int I = 0; I < 8; ++I)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        P[I][t] = Q[I][t];
            }
            last(P);
        } else {
            // (two slots per iteration, so that P and Q swap without copies)
            for (; j >= 1; j -= 2) {
                again = slot(P, Q, j);
                if (again)
                    break;
                again = slot(Q, P, j - 1);
                if (again)
                    break;
            }
            if (!again && j == 0) {
                again = slot(P, Q, 0);
                if (!again)
                    last(Q);
            } else if (!again) {
                last(P);
            }
        }
        if (!again) {
            __syncthreads();
            if (args.progress)
                __syncthreads();
        }
    } else {
        // ---- staging waves --------------------------------------------------
        // chunk i of this thread: row i * 32 + srow, columns 4 sgi .. + 3 of the
        // panel; after the row reduce, lanes 2 i, 2 i + 1 of the eight lanes of
        // a row hold the sum of row i * 32 + srow (the even one owns it)
        const int st = tid - 256, sgi = st & 7, srow = st >> 3;
        const int orow = (sgi >> 1) * 32 + srow;
        const bool oown = (sgi & 1) == 0;
        const int wpos = panel_pos(srow, sgi & 3) + ((sgi >> 2) << 2);  // chunk i adds 1024 i
        // slots loaded ahead: a hinted slot may have one panel and no time in it
        // for the loads of the next one's four
        constexpr int NPF = HINT ? 2 : 1;
        u4 pf[NPF][kNP][4];
        uint32_t pfb = 0;
        // compact storage: offsets of the slot being loaded (A, b) and stored
        // (lambda), each walked down from the chain's end
        int32_t curA = args.totalA, curB = args.totalR, curL = args.totalR;
        // panel q of slot s, of wr row and wc column blocks (rows past the slot's,
        // and slots before the segment, lie outside the resource and read as
        // zero)
        auto load = [&](u4(&dst)[kNP][4], int q, int64_t s, int wr, int wc) {
            const int ld = pitch(wc);
            const int nrow = s >= 0 && q < panels(wc) ? 16 * wr : 0;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(A + (compact ? (int64_t)__builtin_amdgcn_readfirstlane(curA)
                              : (s >= 0 ? s : 0) * (int64_t)(kR * kR))),
                0, __builtin_amdgcn_readfirstlane(nrow * ld * 4), kBufferWord3);
            int off = srow * (ld * 4) + sgi * 16;
            if (compact)
                off |= q * kPC + 4 * sgi < ld ? 0 : kOutOfRange;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                dst[q][i] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + i * 32 * (ld * 4),
                                                                  q * kPC * 4, 0);
        };
        auto load_b = [&](int64_t s, int wr) {
            if constexpr (AFF) {
                const int nrow = s < 0 ? 0 : compact ? 16 * wr : kR;
                if (compact)
                    curB -= nrow;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(bv + (compact ? (int64_t)__builtin_amdgcn_readfirstlane(curB)
                                   : (s >= 0 ? s : 0) * (int64_t)kR)),
                    0, __builtin_amdgcn_readfirstlane(nrow * 4), kBufferWord3);
                pfb = __builtin_amdgcn_raw_buffer_load_b32(rs, orow * 4, 0, 0);
            }
        };
        float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        // panel q of slot s from registers into LDS, and its share of c_s
        int buf = 0;
        // (wq[d]: blocks of slot s + 1 - d, d = 0 .. NPF + 1)
        auto stage = [&](u4(&src)[kNP][4], int q, int64_t s, const int *wq) {
            f4 cv = {};
            if constexpr (AFF)
                cv = *(const f4 *)&sC[(s + 1) & 3][q * kPC + 4 * sgi];
            // (the products read no row blocks past these)
            const int nst = kShapes && s >= 0 ? (wq[1] <= 2 ? 1 : wq[1] <= 4 ? 2 : 4) : 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (kShapes && i >= nst) {
                    part[i] = 0.0f;
                    continue;
                }
                const float x0 = bitsf(src[q][i][0]), x1 = bitsf(src[q][i][1]);
                const float x2 = bitsf(src[q][i][2]), x3 = bitsf(src[q][i][3]);
                if constexpr (AFF) {
                    const float d = x0 * cv[0] + x1 * cv[1] + x2 * cv[2] + x3 * cv[3];
                    part[i] = q == 0 ? d : part[i] + d;
                }
                const Split2 s01 = split_pair(x0, x1), s23 = split_pair(x2, x3);
                __bf16 *dst = sA[HINT ? buf : q & 1] + wpos + 1024 * i;
                *(u2 *)dst = u2{s01.h, s23.h};
                *(u2 *)(dst + kPlane) = u2{s01.m, s23.m};
                *(u2 *)(dst + 2 * kPlane) = u2{s01.l, s23.l};
            }
            buf ^= 1;
            // the registers take panel q of slot s - NPF, and after the last panel
            // of slot s those that slot s did not use
            const bool end = s >= 0 && q == panels(wq[0]) - 1;
            if (compact && q == 0 && s >= NPF)
                curA -= 16 * wq[NPF + 1] * pitch(wq[NPF]);
            load(src, q, s - NPF, wq[NPF + 1], wq[NPF]);
            if (HINT && end) {
#pragma unroll
                for (int u = 1; u < kNP; ++u)
                    if (u > q)
                        load(src, u, s - NPF, wq[NPF + 1], wq[NPF]);
            }
            if constexpr (AFF) {
                if (end) {
                    group_reduce<8, 4>(part, sgi);
                    if (oown)
                        sC[s & 3][orow] = part[0] + bitsf(pfb);
                    load_b(s - 1, wq[2]);
                }
            }
        };
        // lambda_s (or, with composites, c_s), by the first two staging waves
        int32_t pub_left = args.pchunk;
        int64_t pub = -1;  // slots final once the next barrier is passed, or -1
        int64_t npub = 0;  // publications so far
        float row = 0.0f;  // the range check's bound, from slot s + 1
        // (j: the loop's slot, or -1 past it)
        auto finish = [&](int64_t s, int wr, int64_t j) {
            const int nrow = compact ? 16 * wr : kR;
            if (compact)
                curL -= nrow;
            if (st < kR) {
                const float c = AFF ? sC[s & 3][st] : 0.0f;
                if constexpr (OUT == kOutLambda) {
                    float *lam = args.lam + (compact ? beta * (int64_t)args.totalR + curL
                                                     : (first + s) * (int64_t)kR);
                    const float sum = (sPart[s & 1][0][st] + sPart[s & 1][1][st]) +
                                      (sPart[s & 1][2][st] + sPart[s & 1][3][st]);
                    const float p = HINT && st >= 16 * wr ? 0.0f : sum;
                    if (st < nrow)
                        lam[st] = p + c;
                    const float a = fabsf(p + c);
                    if (__builtin_expect(!(a < kFull) || (a > 0.0f && a < row), 0)) {
                        atomicMax(&sWorst, (int32_t)s);
                        if (!HINT && j >= 0)
                            sFound[j & 1] = (int32_t)j;
                    }
                    row = a * kShow;
                } else if (args.cout && (!args.agg_only || s == 0)) {
                    args.cout[(cslot + s) * kR + st] = c;
                }
            }
            // streaming: at a publish point both storing waves make their
            // stores visible device-wide; publish() follows the next barrier
            if constexpr (OUT == kOutLambda) {
                if (args.progress) {
                    if (--pub_left == 0 || s == 0) {
                        pub = K - s;
                        if (st < kR)
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    }
                    if (pub_left == 0)
                        pub_left = args.pchunk;
                }
            }
        };
        // raises the chain's count (system scope: it lands in memory, past this
        // XCD's L2) and records the clock
        auto publish = [&]() {
            if constexpr (OUT == kOutLambda) {
                // (nothing from the slot that shows a loss on)
                if (pub >= 0 && st == 0 && sWorst < 0) {
                    __hip_atomic_fetch_max(&args.progress[beta], (uint32_t)pub, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_SYSTEM);
                    if (args.pub_clock)
                        args.pub_clock[beta * args.npub + npub] = __builtin_amdgcn_s_memrealtime();
                    sNpub = ++npub;
                }
                pub = -1;
            }
        };
        if (compact)
            curA -= 16 * blocks(K - 1) * pitch(blocks(K));
#pragma unroll
        for (int u = 0; u < NPF; ++u) {
            if (compact && K - 2 - u >= 0)
                curA -= 16 * blocks(K - 2 - u) * pitch(blocks(K - 1 - u));
#pragma unroll
            for (int q = 0; q < kNP; ++q)
                load(pf[u], q, K - 2 - u, blocks(K - 2 - u), blocks(K - 1 - u));
        }
        if (AFF && st < kR) {
            const int nrow = compact ? 16 * blocks(K - 1) : kR;
            const float *bl = bv + (compact ? (int64_t)args.totalR - nrow : (K - 1) * (int64_t)kR);
            sC[(K - 1) & 3][st] = st < nrow ? bl[st] : 0.0f;
        }
        if (compact)
            curB -= 16 * blocks(K - 1);
        load_b(K - 2, blocks(K - 2));
        __syncthreads();
        // wq[d]: blocks of slot j + 2 - d in the slot loop below
        int wq[NPF + 4];
#pragma unroll
        for (int d = 0; d < NPF + 4; ++d)
            wq[d] = blocks(K - d);
        stage(pf[0], 0, K - 2, wq + 1);
        // In the phase of panel p of slot j the next panel is staged: the rest of
        // slot j from its registers, the first of slot j - 1 from the others.
        // The slot's first phase also stores lambda_{j+2}: the apply of slot
        // j + 2 ran in slot j + 1, before this phase's barrier.
        auto slot = [&](u4(&cur)[kNP][4], u4(&next)[kNP][4], int64_t j) {
            const int np = panels(wq[1]);
            const int wnext = blocks(j - 2 - NPF);
            int32_t found = -1;
#pragma unroll
            for (int p = 0; p < kNP; ++p) {
                if (HINT && p >= np)
                    break;
                __syncthreads();
                publish();
                if (!HINT && p == 0)
                    found = sFound[(j + 1) & 1];
                if (p + 1 < kNP && p + 1 < np)
                    stage(cur, p + 1 < kNP ? p + 1 : 0, j, wq + 1);
                else
                    stage(next, 0, j - 1, wq + 2);
                if (p == 0 && j + 2 < K)
                    finish(j + 2, wq[0], j);
            }
#pragma unroll
            for (int d = 0; d < NPF + 3; ++d)
                wq[d] = wq[d + 1];
            wq[NPF + 3] = wnext;
            return !HINT && __builtin_amdgcn_readfirstlane(found) == (int32_t)(j + 1);
        };
        for (int64_t j = K - 2; j >= 0 && !again; j -= NPF) {
            again = slot(pf[0], pf[NPF - 1], j);
            if (NPF == 2 && j >= 1)
                slot(pf[NPF - 1], pf[0], j - 1);
        }
        if (!again) {
            __syncthreads();
            publish();
            if (K >= 2)
                finish(1, blocks(1), -1);
            __syncthreads();
            publish();
            finish(0, blocks(0), -1);
            if (args.progress) {
                __syncthreads();
                publish();
            }
        }
    }

    __syncthreads();
    if (__builtin_expect(sWorst >= 0, 0))
        exact_pass<AFF, HINT, OUT, NT>(sWorst, sNpub, &sC[0], &sPart[0]);
}

}  // namespace

hipError_t launch_chain_wide_f32x(const ChainLaunch &c)
{
    void *params[] = {(void *)&c.args};
    // r_K <= 64: P's columns from 64 on are zero, and a matrix wave that holds one column
    // block instead of two has half of the splits, copies and sums beside its products,
    // which is what bounds a slot of few row blocks (the same results: the rest adds
    // exact zeros).  Two blocks / one, us: widths 32/64/128, 1024 x 64, with b 715 / 675,
    // compact without b 693 / 643; width 32, 600 x 64 268 / 235; width 64 652 / 587.  The
    // fp32 matrix cores take 807, 663, 392 and 542 there: chains of no width above 64
    // belong in r = 64 storage.  (Segments end in widths of their own.)
    const bool narrow = c.ncol <= 4 && c.args.S == 1;
    auto pick = [&](auto aff, auto hint) -> const void * {
        constexpr bool AFF = decltype(aff)::value;
        constexpr int HINT = decltype(hint)::value;
        if constexpr (HINT != kHintCompact)
            if (c.out == kOutComposite)
                return (const void *)&scan_wide_kernel<AFF, HINT, kOutComposite, 2>;
        if constexpr (HINT != kHintNone)
            if (narrow)
                return (const void *)&scan_wide_kernel<AFF, HINT, kOutLambda, 1>;
        return (const void *)&scan_wide_kernel<AFF, HINT, kOutLambda, 2>;
    };
    auto form = [&](auto hint) {
        return c.aff ? pick(std::true_type{}, hint) : pick(std::false_type{}, hint);
    };
    const void *f = !c.hint ? form(std::integral_constant<int, kHintNone>{})
                    : c.args.compact ? form(std::integral_constant<int, kHintCompact>{})
                                     : form(std::integral_constant<int, kHintWidths>{});
    return hipLaunchKernel(f, dim3((unsigned)(c.B * c.args.S)), dim3(512), params, 0, c.stream);
}

}  // namespace lbi
