// Dynamic per-token activation quantisation, the step directly upstream of the W4A8 GEMM
// (paper Sec. 6, "Serving System": FP16 activations are divided by the smooth scale and
// mapped to INT8 per token on the fly):
//
//     x'[m,k] = (float)X[m,k] / smooth[k]                (smooth optional)
//     s_x[m]  = max_k |x'[m,k]| / 127                    (1 for an all-zero token)
//     Q[m,k]  = clamp(rint(x'[m,k] / s_x[m]), -127, 127)
//
// Every operation is one correctly rounded FP32 operation, so the INT8 result is determined
// bit for bit; the kernel reproduces it exactly (see div_by and round8 for how the two divisions
// are shortened where that cannot matter).
//
// One block per token (or per R consecutive tokens, one after the other, so that the reciprocals
// of the smooth scales are computed once for R tokens).  A token of up to 32768 elements is read
// from HBM once and kept in registers between the max pass and the rounding pass; longer tokens
// are read twice (the second read hits L2).  Traffic: 2 bytes in, 1 byte out per element.
#include <algorithm>

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "lqq_common.h"
#include "lqq_device.h"

namespace lqq {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// 8 FP16 values (one 16-byte load) -> FP32
__device__ __forceinline__ void widen8(const u32x4 x, float (&f)[8])
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t w = x[d];
        const f16x2 h = __builtin_bit_cast(f16x2, w);
        f[2 * d] = (float)h[0];
        f[2 * d + 1] = (float)h[1];
    }
}

// the smooth scales of piece i (8 columns)
__device__ __forceinline__ void load_smooth8(const float *smooth, int i, float (&s)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(smooth + 8 * (size_t)i);
    const float4 b = *reinterpret_cast<const float4 *>(smooth + 8 * (size_t)i + 4);
    s[0] = a.x, s[1] = a.y, s[2] = a.z, s[3] = a.w;
    s[4] = b.x, s[5] = b.y, s[6] = b.z, s[7] = b.w;
}

// x / s, correctly rounded, for x = the lower (H = 0) or upper half of xx and y = the correctly rounded
// 1 / s: one exact residual corrects the quotient x * y.  For a general x that can miss by one unit;
// for the 11-bit significand of an FP16 x it never does (tests/native/short_division.c goes through
// all 2^23 x 2^10 pairs of significands).  No intermediate leaves the normal range while s is within
// [2^-40, 2^40] (x is zero or 2^-24 .. 65504); callers check that.  The residual of an infinite x is
// not a number: the fix-up instruction that ends the IEEE sequence gives the quotient that x * y then
// is, infinite (NaN for a NaN).  The mixed-precision FMA takes x as it is, which pays for the fix-up
// (4096 x 8192 22.9 us, 22.9 without either, 23.7 with the fix-up and a conversion of x; 8192 x 2056, bound by
// its instructions, 20.6, 20.2 and 21.8).
template <int H>
__device__ __forceinline__ float div_by(uint32_t xx, float s, float y)
{
    float q, r;
    if (H == 0) {
        asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(q) : "v"(xx), "v"(y));
        asm("v_fma_mix_f32 %0, -%1, %2, %3 op_sel_hi:[0,0,1]" : "=v"(r) : "v"(s), "v"(q), "v"(xx));
    } else {
        asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(q) : "v"(xx), "v"(y));
        asm("v_fma_mix_f32 %0, -%1, %2, %3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(r) : "v"(s), "v"(q), "v"(xx));
    }
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(r, y, q), s, q);
}
__device__ __forceinline__ bool short_division_is_exact(float s) { return s >= 0x1p-40f && s <= 0x1p40f; }

__device__ __forceinline__ float max_abs8(const float (&f)[8], float m)
{
#pragma unroll
    for (int e = 0; e < 8; e += 2) m = fmaxf(fmaxf(m, fabsf(f[e])), fabsf(f[e + 1]));
    return m;
}

// Q = clamp(rint(f / s)) for 8 values.  The FP32 quotient is only needed to decide an integer, so
// the common case multiplies by an approximate reciprocal, in one FMA with 1.5 * 2^23: the sum is
// rounded to an integer, which is its low byte.  The exact product and the correctly rounded
// quotient both lie within 127 * (2^-23 + 2^-24) < 2.3e-5 of the exact quotient (|f / s| <= 127,
// reciprocal within one unit), hence they round to the same integer unless the product is within 3e-5
// of a tie.  Only then (or where a value is not finite) that value is redone with the IEEE division,
// so the result is always that of the division.  A wave of 512 values meets one 3 times in 100, and a small call
// lasts as long as its slowest wave, hence a branch for each of the lane's values: redoing all 8 takes 1.02 to 1.06 of the
// time (8000 calls).  Where most values are ties a loop over the lane's, one selected at a time, takes as long on
// Gaussian values and up to twice as long on these (1311 x 27584 of halves 63 us, all 8 35.7, here 36.8).
__device__ __forceinline__ uint2 round8(const float (&f)[8], float s, float rcp_s)
{
    constexpr float kMagic = 0x1.8p23f;
    uint32_t u[8], ties = 0;  // bit e: value e needs the division
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float t = __builtin_fmaf(f[e], rcp_s, kMagic);
        const float off = __builtin_fmaf(f[e], rcp_s, -(t - kMagic));
        ties |= fabsf(off) <= 0.5f - 3e-5f ? 0u : 1u << e;  // (set for NaN)
        u[e] = __builtin_bit_cast(uint32_t, t);
    }
    // (a branch the compiler must not turn into divisions and selects for everybody)
    if (__builtin_expect_with_probability(ties != 0, 0, 0.999)) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (__builtin_expect_with_probability((ties >> e) & 1, 0, 0.999))
                u[e] = (uint32_t)(int)fminf(fmaxf(__builtin_rintf(f[e] / s), -127.0f), 127.0f);
    }
    uint32_t w[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)  // the low bytes of four registers
        w[h] = __builtin_amdgcn_perm(u[4 * h + 1], u[4 * h], 0x0c0c0400u) |
               __builtin_amdgcn_perm(u[4 * h + 3], u[4 * h + 2], 0x04000c0cu);
    return uint2{w[0], w[1]};
}

// maximum (of values >= 0) over the block of NWAVES waves; every thread gets the result
template <int CTRL, int ROWS>
__device__ __forceinline__ float lane_shift_or_0(float m)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, m), CTRL, ROWS, 0xf, ROWS == 0xf));
}
template <int NWAVES>
__device__ __forceinline__ float block_max(float m, float *s_part)
{
    m = fmaxf(m, lane_shift_or_0<0x111, 0xf>(m));  // row_shr 1, 2, 4, 8: lane 15 of each row of 16
    m = fmaxf(m, lane_shift_or_0<0x112, 0xf>(m));
    m = fmaxf(m, lane_shift_or_0<0x114, 0xf>(m));
    m = fmaxf(m, lane_shift_or_0<0x118, 0xf>(m));
    m = fmaxf(m, lane_shift_or_0<0x142, 0xa>(m));  // row_bcast 15, 31: lane 63 of the wave
    m = fmaxf(m, lane_shift_or_0<0x143, 0xc>(m));
    if ((threadIdx.x & 63) == 63) s_part[threadIdx.x >> 6] = m;
    __syncthreads();
    float r = s_part[0];
#pragma unroll
    for (int w = 1; w < NWAVES; ++w) r = fmaxf(r, s_part[w]);
    return r;
}

// Tokens of any length, one per block, read twice.  Loads of a pass are issued four pieces at
// a time, with indices past the end clamped to the last piece and their values ignored, so
// that no load waits behind a branch.
constexpr int kLongThreads = 256;
template <bool SMOOTH>
__global__ __launch_bounds__(kLongThreads) void quantize_act_long_kernel(
    int K, const __half *__restrict__ X, const float *__restrict__ smooth, int8_t *__restrict__ Q,
    float *__restrict__ sx)
{
    __shared__ float s_part[4];
    const int m = blockIdx.x, tid = threadIdx.x;
    const u32x4 *xrow = reinterpret_cast<const u32x4 *>(X + (size_t)m * K);
    uint2 *qrow = reinterpret_cast<uint2 *>(Q + (size_t)m * K);
    const int n8 = K >> 3;
    constexpr int U = 4;  // pieces in flight per thread

    float f[U][8], sm[SMOOTH ? U : 1][8];
    auto load = [&](int i0) {
        u32x4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * kLongThreads, n8 - 1);
            raw[u] = xrow[i];
            if (SMOOTH) load_smooth8(smooth, i, sm[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            widen8(raw[u], f[u]);
            if (SMOOTH) {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[u][e] /= sm[u][e];
            }
        }
    };
    float amax = 0.0f;
    for (int i0 = tid; i0 < n8; i0 += U * kLongThreads) {
        load(i0);
#pragma unroll
        for (int u = 0; u < U; ++u) amax = max_abs8(f[u], amax);  // (a piece read twice changes nothing)
    }
    amax = block_max<4>(amax, s_part);
    const float s = amax > 0.0f ? amax / 127.0f : 1.0f;
    if (tid == 0) sx[m] = s;
    const float rcp_s = __builtin_amdgcn_rcpf(s);
    for (int i0 = tid; i0 < n8; i0 += U * kLongThreads) {
        load(i0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kLongThreads;
            if (i < n8) qrow[i] = round8(f[u], s, rcp_s);
        }
    }
}

// Register-resident tokens (K <= ITERS x NT x 8).  Thread t owns the 16-byte pieces t, t + NT, ...
// of a token, i.e. fixed columns; pieces past the end repeat the last one, which leaves the maximum
// alone, and are not stored.
//   SEVERAL: a block takes R consecutive tokens; the smooth scales and their reciprocals are loaded
//     and computed once, and the loads of the next two tokens are in flight while one is worked on.
//     The loads and stores of that loop are all unconditional (past the end: the last token once
//     more, the last piece once more with the same bytes), so that the compiler can count them and
//     a token waits for its own loads only.
//   Otherwise one token per block, and with lg_shares > 0 a share of its pieces: each of the token's
//     2^lg_shares blocks finds the maximum of the whole token and rounds and stores its part of every
//     thread's ITERS pieces.  These blocks are 8 ids apart, on one XCD, whose L2 then fetches the
//     token once.
// About 10 instructions per element with smooth scales, 6 without; large calls move their bytes at
// the rate of a copy or near it, small ones take the launch, one load and one store.
// Without smooth scales eight waves a SIMD are asked for: 1024 threads of four pieces at 66 registers instead of 63 ran one
// block on a CU instead of two, at up to 1.28 of the time.
template <bool SMOOTH, int ITERS, int NT, bool SEVERAL>
__global__ __launch_bounds__(NT, SMOOTH ? 1 : 8) void quantize_act_rows_kernel(
    int M, int K, int R, int lg_shares, const __half *__restrict__ X, const float *__restrict__ smooth,
    int8_t *__restrict__ Q, float *__restrict__ sx)
{
    __shared__ __attribute__((aligned(16))) float s_part[2][NT / 64];
    const int tid = threadIdx.x;
    const int n8 = K >> 3;
    const int row = (int)blockIdx.x >> 3, share = row & ((1 << lg_shares) - 1);
    const int m_first = SEVERAL ? (int)blockIdx.x * R : (row >> lg_shares) * 8 + ((int)blockIdx.x & 7);
    if (m_first >= M) return;  // (several shares: the grid is padded to 8 tokens)
    const int it_begin = ITERS * share >> lg_shares, it_end = ITERS * (share + 1) >> lg_shares;
    int piece[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) piece[it] = min(it * NT + tid, n8 - 1);
    const int m_begin = m_first, m_end = SEVERAL ? min(M, m_begin + R) : m_begin + 1;

    u32x4 raw[SEVERAL ? 2 : 1][ITERS];  // this token and the next
    auto load = [&](int m, u32x4 (&r)[ITERS]) {
        const u32x4 *xrow = reinterpret_cast<const u32x4 *>(X + (size_t)min(m, m_end - 1) * K);
#pragma unroll
        for (int it = 0; it < ITERS; ++it) r[it] = xrow[piece[it]];
    };
    // (the loads of the first tokens go out before anything waits for the smooth scales)
    load(m_begin, raw[0]);
    if constexpr (SEVERAL) load(m_begin + 1, raw[1]);

    float sm[SMOOTH ? ITERS : 1][8], rc[SMOOTH && SEVERAL ? ITERS : 1][8];
    bool safe = true;  // every smooth scale of this thread allows the short division
    if (SMOOTH) {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            load_smooth8(smooth, piece[it], sm[it]);
            if (SEVERAL) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    rc[SEVERAL ? it : 0][e] = 1.0f / sm[it][e];
                    safe &= short_division_is_exact(sm[it][e]);
                }
            }
        }
    }

    auto token = [&](int m, u32x4 (&r)[ITERS], float *part) {
        float f[ITERS][8];
        float amax = 0.0f;
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            if (SMOOTH && SEVERAL && safe) {
                const float *const y = rc[SEVERAL ? it : 0];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    f[it][2 * d] = div_by<0>(r[it][d], sm[it][2 * d], y[2 * d]);
                    f[it][2 * d + 1] = div_by<1>(r[it][d], sm[it][2 * d + 1], y[2 * d + 1]);
                }
            } else {
                widen8(r[it], f[it]);
                if (SMOOTH) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[it][e] /= sm[it][e];
                }
            }
            amax = max_abs8(f[it], amax);
        }
        if (SEVERAL) load(m + 2, r);
        amax = block_max<NT / 64>(amax, part);
        const float s = amax > 0.0f ? amax / 127.0f : 1.0f;
        if (tid == 0 && share == 0) sx[m] = s;
        const float rcp_s = __builtin_amdgcn_rcpf(s);
        uint2 *qrow = reinterpret_cast<uint2 *>(Q + (size_t)m * K);
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            if (!SEVERAL && (it < it_begin || it >= it_end)) continue;  // (block-uniform)
            const uint2 q = round8(f[it], s, rcp_s);
            if (SEVERAL || it * NT + tid < n8) qrow[piece[it]] = q;
        }
    };
    token(m_begin, raw[0], s_part[0]);
    if constexpr (SEVERAL) {
        for (int m = m_begin + 1; m < m_end; m += 2) {
            token(m, raw[1], s_part[1]);
            if (m + 1 == m_end) break;
            token(m + 1, raw[0], s_part[0]);
        }
    }
}

// (lds: dynamic LDS that nothing uses, to keep fewer blocks on a CU)
template <bool SMOOTH, int ITERS, int NT, bool SEVERAL = false>
static void launch_rows(int M, int K, int R, int lg_shares, const __half *X, const float *smooth, int8_t *Q, float *sx,
                        hipStream_t st, size_t lds = 0)
{
    const int blocks = lg_shares ? ((M + 7) / 8 * 8) << lg_shares : (M + R - 1) / R;
    hipLaunchKernelGGL((quantize_act_rows_kernel<SMOOTH, ITERS, NT, SEVERAL>), dim3((unsigned)blocks), dim3(NT), lds, st, M, K,
                       R, lg_shares, X, smooth, Q, sx);
}

// Block shapes, from sweeps of threads x pieces per thread x tokens per block over M = 4..8192 and
// K = 2048..28672 (microseconds of the rule / of blocks of 256 threads with all pieces of a token, unless said):
//   many tokens, no smooth scales: 256 threads up to 8192 columns (13.3 / 13.5 on 6000 x 4096, 512 threads:
//     15.6), with three pieces each up to 6144 (11.9 on 4096 x 4104, 13.3 on 4096 x 5120; 512 threads of
//     two pieces, nearly half of them past the end: 15.0 and 15.8) and four from there on (18.2 on 4096 x
//     8192, 512 threads: 19.0; with 1024 tokens 7.7 and 7.5, hence from 2048 tokens), one up to 2048 columns
//     (11.0 / 15.5 on 8192 x 2048); 512 threads of three up to 10240 (7880 x 8680 36.0; 768 threads of two, nearly
//     a third of them past the end: 41.1; with 1536 tokens equal, hence from 2048), 768 threads of two pieces up to 12288 (36.8
//     on 6000 x 11008, 512 threads of three: 37.9); 512 threads above (40.2 / 43.5 on 6000 x 14336), three blocks
//     of them on a CU instead of four where the call moves more than the memory-side cache holds (72.3 / 74.5 on
//     8192 x 16384, 62.5 / 64.2 on 8192 x 14336; below that four are ahead, 32.9 / 33.8 on 4096 x 16384);
//   many tokens with smooth scales: from 1024 tokens on several tokens per block, as many as leave two
//     blocks of 1024 threads per CU (one where a thread holds two pieces: 93 registers) -- 18.8 / 26.8
//     on 4096 x 8192 (5.35 TB/s; a copy, which writes as much as it reads, 5.2), 38 / 60 on 4096 x 16384, 9.3 / 11.2 on 1024 x 8192;
//     with at most 2048 columns a token is too short for that (16.0 / 20.2 on 8192 x 2048);
//   few tokens: at most two pieces per thread up to 1536 pieces of a token (45 x 5120 2.64 to 2.30, 200 x 11008
//     4.5 to 3.9 against blocks of 512 threads) and beyond 128 tokens up to 2048 (200 x 14336 5.0 to 4.3); up to
//     64 tokens four blocks, up to 128 two share the pieces of a token (60 x 14336 3.6 to 2.8, 128 x 11008 4.3 to
//     3.2, 16 x 28672 3.1 to 2.9; with 200 tokens two blocks a token are as fast as one, or slower).  These times
//     are what a call adds to a replayed graph behind a kernel that moves 24 MB; an empty kernel adds 1.7.
template <bool SMOOTH>
static void launch_quantize(int M, int K, const __half *X, const float *smooth, int8_t *Q, float *sx, hipStream_t st)
{
    const int n8 = K / 8;  // 16-byte pieces of a token
    if constexpr (SMOOTH) {
        if (M >= 1024 && K > 2048 && K <= 16384) {
            const int R = (M + 511) / 512;
            if (n8 <= 512) return launch_rows<SMOOTH, 1, 512, true>(M, K, R, 0, X, smooth, Q, sx, st);
            if (n8 <= 1024) return launch_rows<SMOOTH, 1, 1024, true>(M, K, R, 0, X, smooth, Q, sx, st);
            return launch_rows<SMOOTH, 2, 1024, true>(M, K, (M + 255) / 256, 0, X, smooth, Q, sx, st);
        }
    }
    const int two = M <= 128 ? 1 : 0, four = M <= 64 ? 2 : two;  // log2 of the blocks that share a token
    if (n8 <= 256) return launch_rows<SMOOTH, 1, 256>(M, K, 1, 0, X, smooth, Q, sx, st);
    if (n8 <= 512)
        return M <= 512 ? launch_rows<SMOOTH, 1, 512>(M, K, 1, 0, X, smooth, Q, sx, st)
                        : launch_rows<SMOOTH, 2, 256>(M, K, 1, 0, X, smooth, Q, sx, st);
    if (n8 <= 768 && (SMOOTH || (M > 128 && M <= 512))) return launch_rows<SMOOTH, 1, 768>(M, K, 1, 0, X, smooth, Q, sx, st);
    if constexpr (!SMOOTH) {
        if (n8 <= 768 && M >= 1024) return launch_rows<SMOOTH, 3, 256>(M, K, 1, 0, X, smooth, Q, sx, st);
        if (n8 <= 1024 && M >= 2048) return launch_rows<SMOOTH, 4, 256>(M, K, 1, 0, X, smooth, Q, sx, st);
        if (n8 > 1024 && n8 <= 1280 && M >= 2048) return launch_rows<SMOOTH, 3, 512>(M, K, 1, 0, X, smooth, Q, sx, st);
        if (n8 > 1536 && n8 <= 2048 && (size_t)M * K >= (96u << 20))
            return launch_rows<SMOOTH, 4, 512>(M, K, 1, 0, X, smooth, Q, sx, st, 48 * 1024);
    }
    if (n8 <= 1024) return launch_rows<SMOOTH, 2, 512>(M, K, 1, two, X, smooth, Q, sx, st);
    if (n8 <= 1536) return launch_rows<SMOOTH, 2, 768>(M, K, 1, two, X, smooth, Q, sx, st);
    if (n8 <= 2048)
        return M > 128 && (SMOOTH || M <= 512) ? launch_rows<SMOOTH, 2, 1024>(M, K, 1, 0, X, smooth, Q, sx, st)
                                               : launch_rows<SMOOTH, 4, 512>(M, K, 1, four, X, smooth, Q, sx, st);
    if (n8 <= 4096) return launch_rows<SMOOTH, 4, 1024>(M, K, 1, four, X, smooth, Q, sx, st);
    hipLaunchKernelGGL((quantize_act_long_kernel<SMOOTH>), dim3((unsigned)M), dim3(kLongThreads), 0, st, K, X, smooth, Q, sx);
}

}  // namespace lqq

using namespace lqq;

extern "C" int w4a8_quantize_activations(int M, int K, const uint16_t *X_f16, const float *smooth,
                                         int8_t *X_i8, float *act_scales, void *hip_stream)
{
    if (M < 0 || K <= 0 || K % 8 != 0 || K > (1 << 24))
        return fail(LQ_ERR_INVALID, "bad shape M=%d K=%d (need M>=0, K>0, K%%8==0)", M, K);
    if (M == 0) return LQ_OK;
    if (!X_f16 || !X_i8 || !act_scales) return fail(LQ_ERR_INVALID, "null pointer");
    const uintptr_t bits = (uintptr_t)X_f16 | (uintptr_t)smooth | (uintptr_t)X_i8 | (uintptr_t)act_scales;
    if (bits & 15) return fail(LQ_ERR_ALIGN, "device pointers must be 16-byte aligned");
    const __half *X = reinterpret_cast<const __half *>(X_f16);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    (void)hipGetLastError();
    // A launch holds fewer than 2^32 threads, and a token takes up to 1024 of them.
    constexpr int kTokensPerLaunch = 1 << 21;
    for (long long m = 0; m < M; m += kTokensPerLaunch) {
        const int rows = (int)std::min<long long>(kTokensPerLaunch, M - m);
        if (smooth)
            launch_quantize<true>(rows, K, X + m * K, smooth, X_i8 + m * K, act_scales + m, st);
        else
            launch_quantize<false>(rows, K, X + m * K, smooth, X_i8 + m * K, act_scales + m, st);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LQ_ERR_HIP, "activation quantisation launch failed: %s", hipGetErrorString(e));
    return LQ_OK;
}
