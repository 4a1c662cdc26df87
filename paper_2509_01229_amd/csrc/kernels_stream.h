// stream16 kernel (M <= 16): weights streamed once, K split between the waves of a block.
// (part of liquidgemm.hip: included there, inside namespace lqq)
#pragma once

// ------------------------------------------------------------------------------------
// stream16 kernel: M <= 16 on v_mfma_i32_16x16x64_i8.  A unit is 128 k (two chunks per tile).  grid =
// (N / (32 F), S): block (bx, ks) owns F tiles and the ks-th of S slices of K; its NW waves take the
// slice's units round-robin.  S > 1 (grid-level split-K) is used when N alone gives too few blocks to
// keep every HBM channel busy; the S partial tiles meet in a workspace and the last block to arrive (a
// ticket per tile group) adds them up and runs the epilogue.  All sums are INT32, so neither level
// of split-K changes the result.
//
// A 32-row MFMA wastes half of its rows on a decode batch, and in this regime the per-CU
// arithmetic (dequantisation + MFMA) is not far below what the HBM stream demands.  The
// packed layout is unchanged: after the usual dequantisation one v_permlane16_swap per
// register turns the chunk's two 32x32x32 operands into the operands of two 16x16x64
// MFMAs (see regroup_16x16), which take half the matrix-pipe time, a quarter of the
// accumulator registers and half of the X registers.
// ------------------------------------------------------------------------------------
// UU = 128-k units per pipeline step (1 or 2): bytes in flight per wave = F * UU * 2 KiB.
template <int F, int UU, bool G128>
struct Stream16Regs {
    u32x4 w[F][2 * UU];
    UnitParams<G128> p[F][UU];
    u32x4 x[2 * UU];
};

template <int F, int NW, int UU, bool G128>
__device__ __forceinline__ void stream16_block(
    const Place pl, int M, int N, int K, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials)
{
    constexpr int VALS = F * 8;  // accumulator registers per lane
    extern __shared__ __attribute__((aligned(16))) int red[];  // [NW][VALS][64]
    __shared__ int s_last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 31;
    const int t0 = pl.gx * F;
    const int units = K >> 7;                   // 128-k units (parameter granularity)
    const int steps = units / UU;               // pipeline steps of UU units
    const int chunks_per_tile = K >> 6;
    const int S = pl.S, ks = pl.ks;
    const int u_begin = (int)((long long)steps * ks / S), u_end = (int)((long long)steps * (ks + 1) / S);

    v4i acc[F][2];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[f][h] = v4i{0, 0, 0, 0};

    // X operand of a 16x16x64 MFMA: lane l supplies row l%16, k-block l/16 of a chunk, in
    // the k-block order that regroup_16x16 produces.  Lanes past M read row M-1.
    const int8_t *xrow = X + (size_t)min(lane & 15, M - 1) * K + kstep16_offset(lane >> 4);

    // The outputs this thread will finish (idx = threadIdx.x + i * blockDim.x) are known
    // now: fetch their scales here, so that the epilogue does not end on a cold load.
    constexpr int OUTS = (VALS * 64 + NW * 64 - 1) / (NW * 64);
    float pre_sx[OUTS], pre_sw[OUTS];
    if (Y) {
#pragma unroll
        for (int i = 0; i < OUTS; ++i) {
            const int idx = threadIdx.x + i * NW * 64;
            const int v = min(idx >> 6, VALS - 1), l = idx & 63;
            pre_sx[i] = sx[min(4 * (l >> 4) + (v & 3), M - 1)];
            pre_sw[i] = sw[channel_of(t0 + (v >> 3), 16 * ((v >> 2) & 1) + (l & 15))];
        }
    }

    auto load_unit = [&](int u, Stream16Regs<F, UU, G128> &r) {
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const u32x4 *base = Wp + ((size_t)(t0 + f) * chunks_per_tile + 2 * UU * (size_t)u) * 64 + lane;
#pragma unroll
            for (int c = 0; c < 2 * UU; ++c) r.w[f][c] = __builtin_nontemporal_load(base + 64 * c);
#pragma unroll
            for (int q = 0; q < UU; ++q) {
                r.p[f][q].load(gp, (size_t)(t0 + f) * units + (size_t)u * UU + q, j);
            }
        }
#pragma unroll
        for (int c = 0; c < 2 * UU; ++c)
            r.x[c] = *reinterpret_cast<const u32x4 *>(xrow + (size_t)u * (128 * UU) + 64 * c);
    };
    auto compute_unit = [&](const Stream16Regs<F, UU, G128> &r) {
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int c = 0; c < 2 * UU; ++c) {
                uint32_t s2, a4;
                r.p[f][c >> 1].get(c & 1, s2, a4);
                v4i lo, hi, b1, b2;
                dequant_chunk(r.w[f][c], s2, a4, lo, hi);
                regroup_16x16(lo, hi, b1, b2);
                const v4i xa = __builtin_bit_cast(v4i, r.x[c]);
                acc[f][0] = mfma16_i8(xa, b1, acc[f][0]);
                acc[f][1] = mfma16_i8(xa, b2, acc[f][1]);
            }
    };

    Stream16Regs<F, UU, G128> cur, nxt;
    int u = u_begin + wave;
    if (u < u_end) load_unit(u, cur);
    for (; u < u_end; u += NW) {
        const bool more = (u + NW) < u_end;
        if (more) load_unit(u + NW, nxt);
        compute_unit(cur);
        if (more) cur = nxt;
    }

    // in-block split-K reduction: value v = (f*2 + h)*4 + r of lane l is row 4*(l/16) + r,
    // slot 16*h + l%16 of tile t0 + f
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wave * VALS + (f * 2 + h) * 4 + r) * 64 + lane] = acc[f][h][r];
    __syncthreads();
    auto block_sum = [&](int idx) {
        int sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += red[(w * VALS + (idx >> 6)) * 64 + (idx & 63)];
        return sum;
    };
    auto finish = [&](int i, int idx, int sum) {
        const int v = idx >> 6, l = idx & 63;
        const int m = 4 * (l >> 4) + (v & 3);
        if (m < M) {
            const int n = channel_of(t0 + (v >> 3), 16 * ((v >> 2) & 1) + (l & 15));
            if (ACC) ACC[(size_t)m * N + n] = sum;
            if (Y) Y[(size_t)m * N + n] = scale_to_half(sum, pre_sx[i], pre_sw[i]);
        }
    };
    if (S == 1) {
#pragma unroll
        for (int i = 0; i < OUTS; ++i) {
            const int idx = threadIdx.x + i * NW * 64;
            if (idx < VALS * 64) finish(i, idx, block_sum(idx));
        }
    } else {
        // Partial tile of this slice: [ks][blockIdx.x][VALS * 64], coalesced.  The tiles are
        // written and read with device-scope atomics, which act at the memory side common to
        // all XCDs, so no cache has to be flushed or invalidated.  Every wave waits for the
        // acknowledgement of its own stores (a block barrier alone does not: it orders LDS
        // traffic only) before the barrier that precedes the ticket, so a block that sees
        // the last ticket also sees every partial tile.
        int32_t *mine = partials + ((size_t)ks * pl.gnx + pl.gx) * (size_t)(VALS * 64);
        for (int idx = threadIdx.x; idx < VALS * 64; idx += NW * 64)
            __hip_atomic_store(mine + idx, block_sum(idx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_vmcnt0();
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned t = __hip_atomic_fetch_add(&pl.tickets[pl.gx], 1u, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
            s_last = (t == (unsigned)(S - 1));
        }
        __syncthreads();
        if (s_last) {
#pragma unroll
            for (int i = 0; i < OUTS; ++i) {
                const int idx = threadIdx.x + i * NW * 64;
                if (idx >= VALS * 64) break;
                int sum = 0;
                for (int k2 = 0; k2 < S; ++k2)
                    sum += __hip_atomic_load(
                        partials + ((size_t)k2 * pl.gnx + pl.gx) * (size_t)(VALS * 64) + idx,
                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                finish(i, idx, sum);
            }
            if (threadIdx.x == 0)
                __hip_atomic_store(&pl.tickets[pl.gx], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int F, int NW, int UU, bool G128>
__global__ __launch_bounds__(NW * 64) void w4a8_stream16_kernel(
    int M, int N, int K, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials,
    unsigned int *__restrict__ tickets)
{
    stream16_block<F, NW, UU, G128>(grid_place(tickets), M, N, K, X, sx, Wp, gp, sw, Y, ACC, partials);
}

