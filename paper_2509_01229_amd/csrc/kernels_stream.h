// stream16 kernels (M <= 16): weights streamed once, K split between the waves of a block.
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

// The waves' accumulators are in red[NW][VALS][64]: sum over the waves, over the K slices where there are
// several, and epilogue.  Value v of lane l is row 4 (l / 16) + v % 4, channel chan(v, l); thread i's outputs are
// idx = 64 v + l = i, i + 64 NW, ...; their scales are in pre_sx and pre_sw.
template <int VALS, int NW, class Chan>
__device__ __forceinline__ void stream16_finish(
    const Place pl, int M, int N, const int *red, const float *pre_sx, const float *pre_sw, Chan chan,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials)
{
    constexpr int OUTS = (VALS * 64 + NW * 64 - 1) / (NW * 64);
    __shared__ int s_last;
    const int S = pl.S, ks = pl.ks;
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
            const int n = chan(v, l);
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
            // (four slices at a time, all loads on the way before the first is added: one after the other each was a
            // trip to memory of its own -- 8 x 1024 x 8448 in two slices 5.2 / 4.8 us)
            int sum[OUTS] = {};
            for (int k0 = 0; k0 < S; k0 += 4) {
                int part[OUTS][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (k0 + q >= S) continue;
                    const int32_t *other = partials + ((size_t)(k0 + q) * pl.gnx + pl.gx) * (size_t)(VALS * 64);
#pragma unroll
                    for (int i = 0; i < OUTS; ++i)
                        part[i][q] = __hip_atomic_load(other + min((int)threadIdx.x + i * NW * 64, VALS * 64 - 1), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (k0 + q >= S) continue;
#pragma unroll
                    for (int i = 0; i < OUTS; ++i) sum[i] += part[i][q];
                }
            }
#pragma unroll
            for (int i = 0; i < OUTS; ++i) {
                const int idx = threadIdx.x + i * NW * 64;
                if (idx < VALS * 64) finish(i, idx, sum[i]);
            }
            if (threadIdx.x == 0)
                __hip_atomic_store(&pl.tickets[pl.gx], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int F, int NW, int UU, bool G128, bool SCALES_FIRST = false>
__device__ __forceinline__ void stream16_block(
    const Place pl, int M, int N, int K, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials)
{
    constexpr int VALS = F * 8;  // accumulator registers per lane
    extern __shared__ __attribute__((aligned(16))) int red[];  // [NW][VALS][64]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 31;
    const int t0 = pl.gx * F;
    const int units = K >> 7;                   // 128-k units (parameter granularity)
    const int steps = units / UU;               // pipeline steps of UU units
    const int chunks_per_tile = K >> 6;
    const int S = pl.S, ks = pl.ks;
    const int u_begin = slice_begin(steps, ks, S), u_end = slice_begin(steps, ks + 1, S);

    v4i acc[F][2];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[f][h] = v4i{0, 0, 0, 0};

    // X operand of a 16x16x64 MFMA: lane l supplies row l%16, k-block l/16 of a chunk, in
    // the k-block order that regroup_16x16 produces.  Lanes past M read row M-1.
    const int8_t *xrow = X + (size_t)min(lane & 15, M - 1) * K + kstep16_offset(lane >> 4);

    // The outputs this thread will finish (idx = threadIdx.x + i * blockDim.x) are known now: their scales
    // are fetched behind the first unit, so that the epilogue does not end on a cold load -- or ahead of it in a grouped launch,
    // where several rounds of blocks share a CU and the scales are what the end of a short block waits for (8 experts of 9 rows on 12480 x
    // 768 12.0 us, behind the first unit 12.7; plain launches 7 x 13824 x 2560 6.7 ahead, 6.3 behind).
    constexpr int OUTS = (VALS * 64 + NW * 64 - 1) / (NW * 64);
    auto chan = [&](int v, int l) { return channel_of(t0 + (v >> 3), 16 * ((v >> 2) & 1) + (l & 15)); };
    float pre_sx[OUTS], pre_sw[OUTS];
    auto load_scales = [&] {
        if (!Y) return;
#pragma unroll
        for (int i = 0; i < OUTS; ++i) {
            const int idx = threadIdx.x + i * NW * 64;
            const int v = min(idx >> 6, VALS - 1), l = idx & 63;
            pre_sx[i] = sx[min(4 * (l >> 4) + (v & 3), M - 1)];
            pre_sw[i] = sw[chan(v, l)];
        }
    };
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
    if (SCALES_FIRST) load_scales();
    if (u < u_end) load_unit(u, cur);
    if (!SCALES_FIRST) load_scales();
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
    stream16_finish<VALS, NW>(pl, M, N, red, pre_sx, pre_sw, chan, Y, ACC, partials);
}

template <int F, int NW, int UU, bool G128>
__global__ __launch_bounds__(NW * 64) void w4a8_stream16_kernel(
    int M, int N, int K, int S, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials,
    unsigned int *__restrict__ tickets)
{
    // (the arguments up to sw, all that the first loads need, come in registers: see w4a8_panel_kernel)
    const Place pl{(int)blockIdx.x, N / (32 * F), (int)blockIdx.y, S, tickets};
    stream16_block<F, NW, UU, G128>(pl, M, N, K, X, sx, Wp, gp, sw, Y, ACC, partials);
}


// ------------------------------------------------------------------------------------
// Half a tile (16 channels) per block: twice the blocks where N alone leaves CUs idle, and no exchange of K
// slices where these would fill them.  Such calls are bound by launch, the latency of the first loads and the sum over the
// waves: 4 x 4096 x 4096 takes 4.2 us (whole tiles 5.1), 4 x 4096 x 11008 7.2 (two slices of K 8.9), 4.3 TB/s with weights
// from HBM.  A unit of 128 k is one 16-byte load per lane: lane l takes slot 16 half + l % 16, k-half (l / 16) % 2, of chunk
// l / 32.  Its low nibbles are then, without any regrouping, the B operand of a 16x16x64 MFMA over the first k-steps of
// both chunks and its high nibbles over the second; X is read in that order.  All loads of D units per wave
// are issued together and twice that are in flight; units past the end are loads past the end of the buffers (zero X, so
// they add nothing), and the waves do not branch on them.
// ------------------------------------------------------------------------------------
template <int D>
struct HalfRegs {
    u32x4 w[D], x[D][2];
    uint32_t p[D];
};

template <int NW, int D, bool G128>
__device__ __forceinline__ void stream16_half_block(
    const Place pl, int M, int N, int K, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials)
{
    __shared__ int red[NW * 4 * 64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tile = pl.gx >> 1, slot = 16 * (pl.gx & 1) + (lane & 15);
    const int chunk = lane >> 5, kb = (lane >> 4) & 1;
    const int units = K >> 7;
    const int u_begin = slice_begin(units, pl.ks, pl.S), u_end = slice_begin(units, pl.ks + 1, pl.S);
    constexpr int PB = G128 ? 64 : 128;  // parameter bytes of a tile's unit
    const buf_t wbuf = make_buf(Wp + (size_t)tile * (K >> 6) * 64, (uint32_t)K * 16u);
    const buf_t pbuf = make_buf(gp + (size_t)tile * units * PB, (uint32_t)units * PB);
    const buf_t xbuf = make_buf(X, (uint32_t)M * (uint32_t)K);
    const uint32_t w_off = 1024 * chunk + 512 * kb + 16 * slot, p_off = slot * (PB / 32);
    const uint32_t x_off = (uint32_t)min(lane & 15, M - 1) * (uint32_t)K + 64 * chunk + 16 * kb;

    auto load = [&](HalfRegs<D> &r, int k0) {  // the wave's units k0 .. k0 + D - 1
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int u = u_begin + wave + (k0 + d) * NW;
            const bool is_unit = u < u_end;
            const int at = is_unit ? u : 0;
            r.w[d] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, is_unit ? w_off : kNoLoad, at * 2048, 2);
            r.p[d] = G128 ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(pbuf, is_unit ? p_off : kNoLoad, at * PB, 0)
                          : __builtin_amdgcn_raw_buffer_load_b32(pbuf, is_unit ? p_off : kNoLoad, at * PB, 0);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                r.x[d][h] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (is_unit ? x_off : kNoLoad) + 32 * h, at * 128, 0);
        }
    };
    v4i acc = {0, 0, 0, 0};
    auto compute = [&](const HalfRegs<D> &r) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            uint32_t s2, a4;
            expand_params(G128 ? r.p[d] : r.p[d] >> (16 * chunk), 0, s2, a4);
            v4i lo, hi;
            dequant_chunk(r.w[d], s2, a4, lo, hi);
            acc = mfma16_i8(__builtin_bit_cast(v4i, r.x[d][0]), lo, acc);
            acc = mfma16_i8(__builtin_bit_cast(v4i, r.x[d][1]), hi, acc);
        }
    };
    const int passes = (u_end - u_begin + NW * D - 1) / (NW * D);  // (the same for every wave)
    HalfRegs<D> a, b;
    auto chan = [&](int, int l) { return channel_of(tile, 16 * (pl.gx & 1) + (l & 15)); };
    float pre_sx = 0, pre_sw = 0;  // (four waves finish one output per thread)
    load(a, 0);
    load(b, D);
    if (Y && threadIdx.x < 256) {
        pre_sx = sx[min(4 * (lane >> 4) + wave, M - 1)];
        pre_sw = sw[chan(0, lane)];
    }
    __builtin_amdgcn_sched_barrier(0);
    int p = 0;
    for (; p + 2 < passes; p += 2) {
        compute(a);
        load(a, (p + 2) * D);
        __builtin_amdgcn_sched_barrier(0);
        compute(b);
        load(b, (p + 3) * D);
        __builtin_amdgcn_sched_barrier(0);
    }
    compute(a);
    if (p + 1 < passes) compute(b);
#pragma unroll
    for (int r = 0; r < 4; ++r) red[(wave * 4 + r) * 64 + lane] = acc[r];
    stream16_finish<4, NW>(pl, M, N, red, &pre_sx, &pre_sw, chan, Y, ACC, partials);
}

template <int NW, int D, bool G128>
__global__ __launch_bounds__(NW * 64) void w4a8_stream16_half_kernel(
    int M, int N, int K, int S, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials,
    unsigned int *__restrict__ tickets)
{
    const Place pl{(int)blockIdx.x, N / 16, (int)blockIdx.y, S, tickets};
    stream16_half_block<NW, D, G128>(pl, M, N, K, X, sx, Wp, gp, sw, Y, ACC, partials);
}
