// panel kernel (17 rows to a few hundred, more with few channels): row tiles of 32 MF rows, K split between the waves of a block.
// (part of liquidgemm.hip: included there, inside namespace lqq)
#pragma once

// ------------------------------------------------------------------------------------
// A block owns 32 MF rows x F tiles (32 F channels) of the output and one of S slices of K; its
// NW waves take the slice's units of 128 k round-robin, so a wave shares nothing with the others
// until the end: no barrier in the loop.  No one unit of the CU is the bound: of 256 x 8192 x 8192 (F = 4, MF = 2) the
// 47.0 thousand cycles that a SIMD's two waves live hold 20.9 of vector and 16.4 of matrix instructions, of 45 x 13824 x
// 5120 (F = 2, MF = 2) the 24.5 hold 7.3 and 5.1 (counters); the form before, with one set of W registers, took 20.6 of 26.5 us and
// 10.2 of 13.7 without its loads, 22.5 and 12.5 without dequantisation and MFMA.  It is the dequantisation of W for few
// rows, the way of X and W to the CU (X in pieces of rows 55 to 60 KB per us and CU also from L2, however many are in flight, whole KiBs 115) and 5 to 7 us of launch,
// first loads and sum, which do not depend on K; hence forms from 1 x 1 to 4 x 4 accumulator tiles, which trade the volume of X and the
// repeated dequantisation against the sum over the waves and the number of blocks.  Two things keep the loads ahead:
//   * W sits in two sets of registers: a unit's is loaded while the unit two before it is computed, as the
//     registers of that one are used up;
//   * X goes straight into LDS, into the half of the wave's region that the unit before the last has left, a
//     whole unit ahead.
// Against one set of W registers (loaded for the next unit) and X through registers, in us: 45 x 5120 x 5120 9.8 / 9.4, 45 x
// 13824 x 5120 14.3 / 13.6, 128 x 4096 x 11008 16.5 / 15.5, 128 x 11008 x 4096 15.0 / 14.4, 24 x 8192 x 4096 7.3 / 6.9, 256 x
// 8192 x 8192 26.7 / 25.6; 18000 calls of 17 to 512 rows 0.96 of the time (groups of 64 and 128 alike), at worst, with K =
// 256, 3.2 / 3.4.
// Starting every column group at another unit takes 1 to 3 us off large batches (35.8 to 32.9 us on 256 x 10240 x
// 8192): rows are a power of two apart, and the blocks of an XCD would all ask the same channels of its L2.
// The sum is one of copies, each wave's in its own region; waves that add to one copy with LDS atomics, each when it is
// through, take longer where K is short (one unit a wave, 32 x 32 6 %, 64 x 64 8 %; 3 x 4 tiles 5 % up to K = 6144) and as long
// where it is not.
// The code is written out per position of a unit (first of an odd count, pair in the loop, last two): a load that
// may or may not have been issued would make the compiler wait for all of them.
//
// X: a load covers 8 whole rows (8 cache lines per KiB instead of the 32 of a fragment load).  Load i (i = 0 .. 4
// MF - 1) fills the 1 KiB piece i of the region in lane order; lane p brings row 8 i + r, 16-byte column c with
// r = (p >> 3) ^ (i & 1), c = (p & 7) ^ r.  Fragment row j' = 32 mf + j is then found in piece j' >> 3
// at 128 ((j & 7) ^ (piece & 1)) + 16 (column ^ (j & 7)): no bank conflict there or in the sum (counted, 0 on both shapes above).
// ------------------------------------------------------------------------------------
// A wave's region holds X of two units, and in the end its sums of up to two tiles.  With one tile and slices in which
// no wave has a second unit half of that does, and short K on many channels has three blocks on a CU instead of
// two (752 blocks of K = 256 5.5 us, with both halves and the sum of one copy 6.9).
constexpr int panel_halves(int F, int NW, int units) { return F == 1 && units <= NW ? 1 : 2; }
constexpr size_t panel_lds_bytes(int F, int NW, int MF, int units)
{
    return (size_t)panel_halves(F, NW, units) * NW * MF * 4096;
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
    extern __shared__ __attribute__((aligned(16))) int8_t panel_lds[];  // the waves' regions: X, then their sums
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j = lane & 31, kb = lane >> 5;
    const int units = K >> 7, tiles = N >> 5;
    const int t0 = pl.gx * F;
    const int m0 = bm * (32 * MF);
    const int S = pl.S, ks = pl.ks;
    const int u_begin = slice_begin(units, ks, S), u_end = slice_begin(units, ks + 1, S);

    v16i acc[F][MF];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][mf][r] = 0;

    const int halves = panel_halves(F, NW, u_end - u_begin);  // (the only one is that of parity 1)
    int8_t *const xregion = panel_lds + wave * (halves * MF * 4096);
    const int8_t *const xfrag = xregion + (j >> 3) * 1024 + 128 * ((j & 7) ^ ((j >> 3) & 1));
    const uint32_t xlds = (uint32_t)(size_t)(__attribute__((address_space(3))) void *)xregion;
    const int rows = min(32 * MF, M - m0);
    const int8_t *const xbase = X + (size_t)m0 * K;
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

    u32x4 wr[2][F][2];  // [parity of the unit]
    std::conditional_t<G128, uint16_t, uint32_t> pr[2][F];  // (widened where it is used: where it is loaded that would wait for it)
    // X of unit u straight into the half of the wave's region for parity `par`
    auto load_x = [&](int u, int par) {
#pragma unroll
        for (int i = 0; i < 4 * MF; ++i)
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                         :
                         : "v"(xoff[i]), "s"(xbase + (size_t)u * 128), "s"(xlds + (1 - par) * (MF * 4096) + i * 1024)
                         : "memory", "m0");
    };
    // (off: the lane's offset, or kNoLoad)
    auto load_w = [&](int u, int par, int f, int c, uint32_t off) {
        wr[par][f][c] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, off + 1024 * c, (min(f, nf - 1) * units + u) * 2048, ONCE ? 2 : 0);
    };
    auto load_p = [&](int u, int par, int f, uint32_t off) {
        const int po = (min(f, nf - 1) * units + u) * PB;
        if constexpr (G128)
            pr[par][f] = __builtin_amdgcn_raw_buffer_load_b16(pbuf, off, po, 0);
        else
            pr[par][f] = __builtin_amdgcn_raw_buffer_load_b32(pbuf, off, po, 0);
    };
    auto load_unit_w = [&](int u, int par, uint32_t w_off, uint32_t p_off) {
#pragma unroll
        for (int f = 0; f < F; ++f) load_p(u, par, f, p_off), load_w(u, par, f, 0, w_off);
#pragma unroll
        for (int f = 0; f < F; ++f) load_w(u, par, f, 1, w_off);
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
    // The units of this wave are wave + k NW of the slice (in an order that starts elsewhere for every column
    // group), k = 0 .. count - 1; only the last may be past the end (is_unit).
    const int n = u_end - u_begin, rot = (int)(((unsigned)pl.gx * NW) % (unsigned)n);
    auto is_unit = [&](int k) { return wave + k * NW < n; };
    auto nth = [&](int k) {
        const int i = min(wave + k * NW, n - 1);
        return u_begin + i + rot - (i + rot >= n ? n : 0);
    };
    // Unit k in 4 F steps of one k-step (32 k) and tile each: the B operand of the next step is
    // dequantised and, at the first tile of a k-step, the X fragments of the next k-step are read
    // while the MFMAs of this one run.  On entry the loads of this unit's W, then its X, then the next
    // unit's W (3 F loads) are in flight.  X of the next unit is loaded at the start, the W registers are loaded
    // again (MORE_W), from unit k + 2, as soon as they are used up.
    auto unit = [&](auto par_tag, auto pending_tag, auto more_w_tag, int k) {
        constexpr int P = decltype(par_tag)::value;
        constexpr bool MORE_W = decltype(more_w_tag)::value, LAST = P == 1 && !MORE_W;
        v4i a[2][MF], b[2];
        uint32_t s2[F], a4[F];
        auto read_a = [&](int t, v4i (&to)[MF]) {
#pragma unroll
            for (int mf = 0; mf < MF; ++mf)
                to[mf] = *reinterpret_cast<const v4i *>(xfrag + ((1 - P) * MF + mf) * 4096 + 16 * ((2 * t + kb) ^ (j & 7)));
        };
        // phase ph (0..3) of the dequantisation of step (t, f): four independent instructions each
        auto build = [&](int t, int f, int ph, v4i &to) {
            if (ph == 0 && (G128 ? t == 0 : (t & 1) == 0)) {
                UnitParams<G128> p;
                p.raw = pr[P][f];
                p.get(t >> 1, s2[f], a4[f]);
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                if (ph == 0) to[d] = (int)((t & 1) ? wr[P][f][t >> 1][d] >> 4 : wr[P][f][t >> 1][d] & 0x0F0F0F0Fu);
                if (ph == 1 && (t & 1)) to[d] &= 0x0F0F0F0F;
                if (ph == 2) to[d] = (int)pk_mad_u16((uint32_t)to[d], s2[f], a4[f]);
                if (ph == 3) to[d] ^= (int)0x80808080;
            }
        };
        // X of this unit is in LDS, and W (older) in the registers
        wait_vmcnt<decltype(pending_tag)::value>();
#pragma unroll
        for (int f = 0; f < F; ++f) asm volatile("" : "+v"(wr[P][f][0]), "+v"(wr[P][f][1]), "+v"(pr[P][f]));
        if (F * MF == 16) {  // (all accumulation registers: held where they are, a copy would need more)
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int mf = 0; mf < MF; ++mf) asm volatile("" : "+a"(acc[f][mf]));
        }
        if (LAST) {
            if (Y) load_scales();
        } else if (is_unit(k + 1)) {
            load_x(nth(k + 1), P ^ 1);
        }
        const int next2 = nth(k + 2);
        const uint32_t w_off = is_unit(k + 2) ? wl : kNoLoad, p_off = is_unit(k + 2) ? pofl : kNoLoad;
        read_a(0, a[0]);
#pragma unroll
        for (int ph = 0; ph < 4; ++ph) build(0, 0, ph, b[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < 4 * F; ++st) {
            const int t = st / F, f = st % F;
            v4i &to = b[(st + 1) & 1];
            if (f == 0 && t < 3) read_a(t + 1, a[(t + 1) & 1]);
#pragma unroll
            for (int mf = 0; mf < MF; ++mf) {
                acc[f][mf] = mfma_i8(a[t & 1][mf], b[st & 1], acc[f][mf]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ph = 4 * mf / MF; ph < 4 * (mf + 1) / MF; ++ph)
                    if (st + 1 < 4 * F) build((st + 1) / F, (st + 1) % F, ph, to);
                // (complete before the registers it comes from are loaded again: these then stay the same ones)
                asm volatile("" : "+v"(to));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (MORE_W && (t & 1)) load_w(next2, P, f, t >> 1, w_off);  // (the B operand of this step was their last use)
            if (MORE_W && t == 3) load_p(next2, P, f, p_off);
        }
    };

    // (an odd count: unit 0 goes first, on the second set of registers)
    const int count = (n + NW - 1) / NW, odd = count & 1;
    if (is_unit(0)) load_x(nth(0), odd);
    if (count > 1) load_unit_w(nth(odd), 0, is_unit(odd) ? wl : kNoLoad, is_unit(odd) ? pofl : kNoLoad);
    load_unit_w(nth(odd ^ 1), 1, is_unit(odd ^ 1) ? wl : kNoLoad, is_unit(odd ^ 1) ? pofl : kNoLoad);
    __builtin_amdgcn_sched_barrier(0);
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    const std::integral_constant<int, 3 * F> next_w{};
    if (odd && count > 1) unit(c1, c0, std::true_type{}, 0);
    for (int k = odd; k + 2 < count; k += 2) {
        unit(c0, next_w, std::true_type{}, k);
        unit(c1, next_w, std::true_type{}, k + 1);
    }
    if (count > 1) unit(c0, next_w, std::false_type{}, count - 2);
    if (is_unit(count - 1))
        unit(c1, c0, std::false_type{}, count - 1);
    else if (Y)
        load_scales();
    __builtin_amdgcn_sched_barrier(0);

    // Sum over the waves through LDS, FG tiles at a time, each wave's in its own region (its reads of X are done).
    // Element quadruple q of (tile, fragment) is 16 bytes per lane: item it = (mf * 4 + q) * 64 + lane of a tile is
    // rows 32 mf + 8 q + 4 (lane / 32) + 0..3 of the slot lane % 32.
    constexpr int FG = F % 2 == 0 ? 2 : 1;
    v4i *const red = reinterpret_cast<v4i *>(panel_lds);
    v4i sums[F][PER];
#pragma unroll
    for (int f0 = 0; f0 < F; f0 += FG) {
        if (f0) __syncthreads();
#pragma unroll
        for (int g = 0; g < FG; ++g)
#pragma unroll
            for (int mf = 0; mf < MF; ++mf)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v16i &t = acc[f0 + g][mf];
                    red[(wave * halves + g) * ITEMS + (mf * 4 + q) * 64 + lane] =
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
                    for (int w = 0; w < NW; ++w) s += red[(w * halves + g) * ITEMS + it];
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
        int *const s_last = reinterpret_cast<int *>(panel_lds);  // (the sums are read before the barrier below)
        wait_vmcnt0();
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned t = __hip_atomic_fetch_add(&pl.tickets[tile_group], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *s_last = (t == (unsigned)(S - 1));
        }
        __syncthreads();
        if (!*s_last) return;
        // Up to three slices at a time (as far as there are registers), all their loads on the way before the first is added: one after the other each
        // was a trip to memory of its own (24 x 4096 x 16384 in four slices 12.8 / 12.3 us).
        constexpr int AT = F * PER >= 8 ? 1 : 3;
        for (int k0 = 1; k0 < S; k0 += AT) {
            unsigned long long v[AT][F][PER][2];
#pragma unroll
            for (int q = 0; q < AT; ++q) {
                if (k0 + q >= S) continue;
                const int k2 = ks + k0 + q - (ks + k0 + q >= S ? S : 0);
                const unsigned long long *other = reinterpret_cast<const unsigned long long *>(base + k2 * group_ints);
#pragma unroll
                for (int f = 0; f < F; ++f)
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        const int it = min((int)threadIdx.x + i * NW * 64, ITEMS - 1);
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            v[q][f][i][h] = __hip_atomic_load(other + (size_t)(f * ITEMS + it) * 2 + h, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT);
                    }
            }
#pragma unroll
            for (int q = 0; q < AT; ++q) {
                if (k0 + q >= S) continue;
#pragma unroll
                for (int f = 0; f < F; ++f)
#pragma unroll
                    for (int i = 0; i < PER; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            sums[f][i][2 * h] += (int)(uint32_t)v[q][f][i][h];
                            sums[f][i][2 * h + 1] += (int)(uint32_t)(v[q][f][i][h] >> 32);
                        }
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

constexpr int kMaxPanelSlices = 64;  // (the dispatcher takes up to 4)

template <int F, int NW, int MF, bool G128, bool ONCE>
__global__ __launch_bounds__(NW * 64) void w4a8_panel_kernel(
    int M, int N, int K, int S, const int8_t *__restrict__ X, const float *__restrict__ sx,
    const u32x4 *__restrict__ Wp, const uint8_t *__restrict__ gp, const float *__restrict__ sw,
    __half *__restrict__ Y, int32_t *__restrict__ ACC, int32_t *__restrict__ partials,
    unsigned int *__restrict__ tickets)
{
    // The command processor hands over the first 14 dwords of the arguments in registers (build.py), as far as `sw`; the first load
    // from the others waits for memory.  So nothing that the first addresses need is taken from those: the row tiles and column
    // groups follow from M and N (us without / with this, 64 x 8192 x 8192 13.8 / 13.5, 45 x 5120 x 13824 14.6 / 14.5, 128 x 11008 x
    // 4096 14.4 / 14.0).  Divisions only where there is something to divide.
    // N is a multiple of 64, so a group of an even number of tiles has an even number of them too: less to clamp in the loop of slices and where the
    // scales are loaded (0.995 of the time with F = 2, 0.999 with 4 over 14000 calls; with F = 1 and 3, where it only moves code, 1.002).
    if constexpr (F % 2 == 0) __builtin_assume((N & 63) == 0 && S >= 1 && S <= kMaxPanelSlices);
    const int blocks_m = (int)(((unsigned)M + 32 * MF - 1) / (32 * MF)), blocks_n = (int)(((unsigned)N / 32 + F - 1) / F);
    // Consecutive block ids go to different XCDs: each XCD gets a run of logical ids, whose row tiles
    // of one column group are neighbours and find its weights in that XCD's L2 (and the slices of a tile end together).
    const int total = blocks_m * blocks_n * S;
    const int xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
    const int lid = xcd * per + min(xcd, rem) + (int)(blockIdx.x >> 3);
    const int tg = S == 1 ? lid : (int)((unsigned)lid / (unsigned)S);
    const int gx = blocks_m == 1 ? tg : (int)((unsigned)tg / (unsigned)blocks_m);
    panel_block<F, NW, MF, G128, ONCE>(Place{gx, blocks_n, lid - tg * S, S, tickets}, tg - gx * blocks_m, M, N, K, X, sx, Wp, gp,
                                       sw, Y, ACC, partials, tg);
}
