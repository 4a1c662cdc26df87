// panel kernel (17 rows to a few hundred, more with few channels): row tiles of 32 MF rows, K split between the waves of a block.
// (part of liquidgemm.hip: included there, inside namespace lqq)
#pragma once

// ------------------------------------------------------------------------------------
// A block owns 32 MF rows x F tiles (32 F channels) of the output and one of S slices of K; its
// NW waves take the slice's units of 128 k round-robin, so a wave shares nothing with the others
// until the end: no barrier in the loop, and the registers of the whole CU hold loads in flight
// (128 KB with F = 4, MF = 2).  Loading further ahead gained nothing (one to four units, F = 1).  Shader
// counters: on 256 x 8192 x 8192 (F = 4, MF = 2, 256 blocks) vector and matrix instructions add up to
// 37.6 of the 51.3 thousand cycles that the two waves of a SIMD live, on 45 x 13824 x 5120 (F = 2, MF = 2, 216
// blocks) 12.8 of 25.6; the waves wait for loads 31 and 37 % of their time, at 21 and 16 bytes per
// cycle and CU (L2 answers in 390 and 480 cycles).  So no one unit is the bound: the dequantisation of W
// for few rows and the latency of X and W both are, hence forms from 1 x 1 to 4 x 4 accumulator tiles, which
// trade the volume of X and the repeated dequantisation against the sum over the waves at
// the end (0.6 us per tile) and the number of blocks.  Starting every column group at another
// unit takes 1 to 3 us off large batches (35.8 to 32.9 us on 256 x 10240 x 8192): rows are a power of
// two apart, and the blocks of an XCD would all ask the same channels of its L2.
// Measured with the dispatcher's choice, before and after, in us: 45 x 13824 x 5120 17.4 / 14.2,
// 45 x 5120 x 13824 20.8 / 16.1, 128 x 11008 x 4096 18.5 / 15.2, 128 x 4096 x 11008 21.2 / 15.8,
// 256 x 8192 x 8192 30.6 / 27.2, 24 x 10240 x 8192 17.1 / 13.6.
//
// X goes through a region of LDS that belongs to the wave: a load covers 8 whole rows (8 cache
// lines per KiB instead of the 32 of a fragment load).  Load i (i = 0 .. 4 MF - 1) fills the 1 KiB
// piece i of the region in lane order; lane p brings row 8 i + r, 16-byte column c with
// r = (p >> 3) ^ (i & 1), c = (p & 7) ^ r.  Fragment row j' = 32 mf + j is then found in piece j' >> 3
// at 128 ((j & 7) ^ (piece & 1)) + 16 (column ^ (j & 7)): neither the stores nor the fragment reads
// meet bank conflicts (the counter says 0 for both shapes above).
// ------------------------------------------------------------------------------------
typedef __amdgpu_buffer_rsrc_t buf_t;
__device__ __forceinline__ buf_t make_buf(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

// ONCE = the weights are read by one row tile only (M <= 32 MF): loaded without keeping them in the
// caches.  That pays where the weights come from HBM, as those of a model larger than the memory-side cache (256 MB)
// do: with 550 MB of weights in rotation 4 to 13 % over 23 shapes of 0.5 to 117 MB at 17..64 rows (1024 x 2048 at 17
// rows 4.5 against 5.1 us, 10240 x 8192 12.9 / 13.7, 28672 x 8192 at 64 rows 30.7 / 32.3; 6144 x 16384 equal).  It
// costs where that cache still holds them all when they are asked for again: 9 to 14 % on 24 matrices of 4096 x
// 4096 in turn (6.9 / 6.1 us at 32 rows), nothing on one matrix of up to 25 MB, up to 17 % on a larger one
// (10240 x 8192 11.9 / 10.9, 28672 x 8192 24.0 / 21.9).  Where row tiles share the weights the plain loads
// win (16 experts of 18..36 rows on 2816 x 2048 16.8 against 18.6).
template <int F, int NW, int MF, bool G128, bool ONCE>
__device__ __forceinline__ void panel_block(
    const Place pl, int bm, int M, int N, int K, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials, int tile_group)
{
    extern __shared__ __attribute__((aligned(16))) int8_t panel_lds[];  // the waves' X regions, then the reduction
    __shared__ int s_last;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j = lane & 31, kb = lane >> 5;
    const int units = K >> 7, tiles = N >> 5;
    const int t0 = pl.gx * F;
    const int m0 = bm * (32 * MF);
    const int S = pl.S, ks = pl.ks;
    const int u_begin = (int)((long long)units * ks / S), u_end = (int)((long long)units * (ks + 1) / S);

    v16i acc[F][MF];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][mf][r] = 0;

    int8_t *const xregion = panel_lds + wave * (MF * 4096);
    const int8_t *const xfrag = xregion + (j >> 3) * 1024 + 128 * ((j & 7) ^ ((j >> 3) & 1));
    const int rows = min(32 * MF, M - m0);
    const buf_t xbuf = make_buf(X + (size_t)m0 * K, (uint32_t)rows * (uint32_t)K);
    uint32_t xoff[4 * MF];
#pragma unroll
    for (int i = 0; i < 4 * MF; ++i) {
        const int r = (lane >> 3) ^ (i & 1), c = (lane & 7) ^ r;
        xoff[i] = (uint32_t)min(8 * i + r, rows - 1) * (uint32_t)K + 16 * c;
    }
    constexpr int PB = G128 ? 64 : 128;  // parameter bytes of a tile's unit
    const int nf = min(F, tiles - t0);   // (tiles past the last repeat it and are not stored)
    const buf_t wbuf = make_buf(Wp + (size_t)t0 * (K >> 6) * 64, (uint32_t)nf * (uint32_t)K * 16u);
    const buf_t pbuf = make_buf(gp + (size_t)t0 * units * PB, (uint32_t)nf * (uint32_t)units * PB);
    const uint32_t wl = lane * 16, pofl = j * (PB / 32);

    u32x4 xr[4 * MF], wr[F][2];
    uint32_t pr[F];
    auto load_x = [&](int u) {
#pragma unroll
        for (int i = 0; i < 4 * MF; ++i) xr[i] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, xoff[i], u * 128, 0);
    };
    auto load_w = [&](int u, int f, int c) {
        wr[f][c] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, wl + 1024 * c, (min(f, nf - 1) * units + u) * 2048, ONCE ? 2 : 0);
    };
    auto load_p = [&](int u, int f) {
        const int po = (min(f, nf - 1) * units + u) * PB;
        pr[f] = G128 ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(pbuf, pofl, po, 0)
                     : __builtin_amdgcn_raw_buffer_load_b32(pbuf, pofl, po, 0);
    };
    // One unit in 4 F steps of one k-step (32 k) and tile each: the B operand of the next step is
    // dequantised and, at the first tile of a k-step, the X fragments of the next k-step are read
    // while the MFMAs of this one run.  MORE: the registers are loaded again, from unit `next`, as
    // soon as they are used up.
    auto unit = [&](auto more_tag, int next) {
        constexpr bool MORE = decltype(more_tag)::value;
        v4i a[2][MF], b[2];
        uint32_t s2[F], a4[F];
        auto read_a = [&](int t, v4i (&to)[MF]) {
#pragma unroll
            for (int mf = 0; mf < MF; ++mf)
                to[mf] = *reinterpret_cast<const v4i *>(xfrag + mf * 4096 + 16 * ((2 * t + kb) ^ (j & 7)));
        };
        auto build = [&](int t, int f, v4i &to) {
            if (G128 ? t == 0 : (t & 1) == 0) {
                UnitParams<G128> p;
                p.raw = pr[f];
                p.get(t >> 1, s2[f], a4[f]);
            }
            dequant_half(wr[f][t >> 1], s2[f], a4[f], t & 1, to);
        };
#pragma unroll
        for (int i = 0; i < 4 * MF; ++i) *reinterpret_cast<u32x4 *>(xregion + i * 1024 + 16 * lane) = xr[i];
        if (MORE) load_x(next);
        read_a(0, a[0]);
        build(0, 0, b[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < 4 * F; ++st) {
            const int t = st / F, f = st % F;
            if (f == 0 && t < 3) read_a(t + 1, a[(t + 1) & 1]);
            if (st + 1 < 4 * F) build((st + 1) / F, (st + 1) % F, b[(st + 1) & 1]);
            if (MORE && (t & 1)) load_w(next, f, t >> 1);  // (the B operand of this step was their last use)
            if (MORE && t == 3) load_p(next, f);
#pragma unroll
            for (int mf = 0; mf < MF; ++mf) acc[f][mf] = mfma_i8(a[t & 1][mf], b[st & 1], acc[f][mf]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // the scales that this thread's outputs need, fetched before its last unit
    constexpr int ITEMS = MF * 4 * 64, PER = (ITEMS + NW * 64 - 1) / (NW * 64);
    float pre_sx[PER][4], pre_sw[F];
    auto load_scales = [&] {
#pragma unroll
        for (int f = 0; f < F; ++f) pre_sw[f] = sw[channel_of(min(t0 + f, tiles - 1), j)];
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) pre_sx[i][e] = sx[min(m0 + 8 * ((wave + i * NW) % (MF * 4)) + 4 * kb + e, M - 1)];
    };
    // unit i of the slice, in an order that starts elsewhere for every column group
    const int n = u_end - u_begin, rot = (int)(((unsigned)pl.gx * NW) % (unsigned)n);
    auto nth = [&](int i) { return u_begin + i + rot - (i + rot >= n ? n : 0); };
    int i = wave;
    if (i < n) {
        const int u = nth(i);
        load_x(u);
#pragma unroll
        for (int f = 0; f < F; ++f) load_p(u, f), load_w(u, f, 0);
#pragma unroll
        for (int f = 0; f < F; ++f) load_w(u, f, 1);
        __builtin_amdgcn_sched_barrier(0);
        for (; i + NW < n; i += NW) unit(std::true_type{}, nth(i + NW));
    }
    if (Y) load_scales();
    __builtin_amdgcn_sched_barrier(0);
    if (i < n) unit(std::false_type{}, 0);

    // Sum over the waves through LDS, FG tiles at a time: element quadruple q of (tile, fragment) as 16
    // bytes per lane.  Item it = (mf * 4 + q) * 64 + lane of a tile is rows 32 mf + 8 q + 4 (lane / 32)
    // + 0..3 of the slot lane % 32.
    constexpr int FG = F % 2 == 0 ? 2 : 1;
    v4i *const red = reinterpret_cast<v4i *>(panel_lds);  // [NW][FG][ITEMS]
    v4i sums[F][PER];
#pragma unroll
    for (int f0 = 0; f0 < F; f0 += FG) {
        __syncthreads();
#pragma unroll
        for (int g = 0; g < FG; ++g)
#pragma unroll
            for (int mf = 0; mf < MF; ++mf)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v16i &t = acc[f0 + g][mf];
                    red[(wave * FG + g) * ITEMS + (mf * 4 + q) * 64 + lane] =
                        v4i{t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]};
                }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < FG; ++g)
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int it = threadIdx.x + i * NW * 64;
                v4i s = {0, 0, 0, 0};
                if (it < ITEMS) {
#pragma unroll
                    for (int w = 0; w < NW; ++w) s += red[(w * FG + g) * ITEMS + it];
                }
                sums[f0 + g][i] = s;
            }
    }
    if (S > 1) {
        // the partial tiles meet in memory: same protocol as stream16_block, 16 bytes per thread
        const size_t group_ints = (size_t)F * ITEMS * 4;
        int32_t *const base = partials + (size_t)tile_group * S * group_ints;
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int it = threadIdx.x + i * NW * 64;
                if (it < ITEMS) store_sc1_x4(base + ks * group_ints + (size_t)(f * ITEMS + it) * 4, sums[f][i]);
            }
        wait_vmcnt0();
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned t = __hip_atomic_fetch_add(&pl.tickets[tile_group], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = (t == (unsigned)(S - 1));
        }
        __syncthreads();
        if (!s_last) return;
        for (int k2 = 0; k2 < S; ++k2) {
            if (k2 == ks) continue;
            const unsigned long long *other = reinterpret_cast<const unsigned long long *>(base + k2 * group_ints);
            unsigned long long v[F][PER][2];
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int it = min((int)threadIdx.x + i * NW * 64, ITEMS - 1);
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        v[f][i][h] = __hip_atomic_load(other + (size_t)(f * ITEMS + it) * 2 + h, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int i = 0; i < PER; ++i)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        sums[f][i][2 * h] += (int)(uint32_t)v[f][i][h];
                        sums[f][i][2 * h + 1] += (int)(uint32_t)(v[f][i][h] >> 32);
                    }
        }
        if (threadIdx.x == 0)  // ready for the next call
            __hip_atomic_store(&pl.tickets[tile_group], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // epilogue (Sec. 4, Sec. 5.3); an even F starts on an even tile, two tiles give adjacent channels
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int it = threadIdx.x + i * NW * 64;
        const int mr = m0 + 8 * (it >> 6) + 4 * kb;
        if (it < ITEMS) {
#pragma unroll
            for (int f = 0; f < F; f += FG) {
                if (f >= nf) continue;
                const int n = channel_of(t0 + f, j);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (mr + e >= M) continue;
                    const size_t o = (size_t)(mr + e) * N + n;
                    if (FG == 2) {
                        if (ACC) *reinterpret_cast<int2 *>(ACC + o) = int2{sums[f][i][e], sums[f + 1][i][e]};
                        if (Y)
                            *reinterpret_cast<__half2 *>(Y + o) =
                                __half2{scale_to_half(sums[f][i][e], pre_sx[i][e], pre_sw[f]),
                                        scale_to_half(sums[f + 1][i][e], pre_sx[i][e], pre_sw[f + 1])};
                    } else {
                        if (ACC) ACC[o] = sums[f][i][e];
                        if (Y) Y[o] = scale_to_half(sums[f][i][e], pre_sx[i][e], pre_sw[f]);
                    }
                }
            }
        }
    }
}

template <int F, int NW, int MF, bool G128, bool ONCE>
__global__ __launch_bounds__(NW * 64) void w4a8_panel_kernel(
    int M, int N, int K, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials,
    unsigned int *__restrict__ tickets, int blocks_m, int blocks_n, int S)
{
    // Consecutive block ids go to different XCDs: each XCD gets a run of logical ids, whose row tiles
    // of one column group are neighbours and find its weights in that XCD's L2.
    const int total = blocks_m * blocks_n * S;
    const int xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
    const int lid = xcd * per + min(xcd, rem) + (int)(blockIdx.x >> 3);
    const int tg = lid / S, ks = lid % S;
    panel_block<F, NW, MF, G128, ONCE>(Place{tg / blocks_m, blocks_n, ks, S, tickets}, tg % blocks_m, M, N, K, X, sx, Wp, gp,
                                       sw, Y, ACC, partials, tg);
}
