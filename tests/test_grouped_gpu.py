"""GPU parity of the grouped (mixture-of-experts) W4A8 GEMM against the CPU oracle: INT32
accumulators bit for bit, FP16 outputs within one ulp, for mixes of expert sizes that reach
all three kernel families, empty experts, ragged tails, and the limits of the interface."""
import sys

import numpy as np
import pytest

from oracle import lqq_oracle as O
from paper_2509_01229_amd import api
from paper_2509_01229_amd import workloads as WL

import gpu_helpers as H
import inputs as I

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


class Experts:
    def __init__(self, E, N, K, g, seed):
        import torch

        self.E, self.N, self.K, self.g = E, N, K, g
        Ws = [WL.make_weights(N, K, 0.02, seed=seed + e) for e in range(E)]
        packs = [api.liquidquant_pack_weights(W, g) for W in Ws]
        self.oracle = [O.quantize_weights(W, g) for W in Ws]
        self.d_packed = torch.from_numpy(np.concatenate([p[0] for p in packs])).cuda()
        self.d_gparams = torch.from_numpy(np.concatenate([p[1] for p in packs])).cuda()
        self.w_scales = np.stack([p[2] for p in packs])
        self.d_w_scales = torch.from_numpy(self.w_scales).cuda()

    def check(self, rows, seed, what):
        import torch

        offs = np.concatenate([[0], np.cumsum(rows)]).astype(int)
        M = int(offs[-1])
        X, s_x = I.make_activations(M, self.K, outlier_frac=0.01, seed=seed)
        ACC_ref, _ = O.grouped_w4a8_gemm(X, s_x, offs, self.oracle)
        s_w_rows = np.concatenate([np.repeat(self.oracle[e]["s_w"][None, :], rows[e], axis=0)
                                   for e in range(self.E)]) if M else np.zeros((0, self.N), np.float32)
        ref64 = ACC_ref.astype(np.float64) * s_x.astype(np.float64)[:, None] * s_w_rows.astype(np.float64)
        dX, dsx = torch.from_numpy(X).cuda(), torch.from_numpy(s_x).cuda()
        Y, ACC = api.w4a8_grouped_gemm(offs, dX, dsx, self.d_packed, self.d_gparams, self.d_w_scales,
                                       self.N, self.K, self.g, want_y=True, want_acc=True)
        torch.cuda.synchronize()
        assert np.array_equal(ACC.cpu().numpy(), ACC_ref), f"{what}: INT32 accumulators differ"
        H.assert_fp16_close(Y.cpu().numpy(), ref64, what)
        return dX, dsx, offs, ACC


CASES = [
    # E, N, K, g, rows per expert
    (5, 256, 512, 64, [3, 0, 20, 40, 200]),        # panels, tiles and an empty expert
    (8, 448, 768, 128, [1, 16, 7, 0, 2, 16, 9, 4]),  # decode-like: every expert small
    (3, 320, 1024, 64, [130, 77, 300]),            # only tiled experts, ragged rows, N tail
    (4, 128, 256, 64, [32, 17, 33, 31]),           # around the family boundaries, one k unit
    (2, 64, 2048, 128, [0, 5]),                    # smallest N, leading empty expert
    # wide layers with many experts: large grids in every family
    (4, 16384, 256, 64, [20, 64, 33, 50]),
    (8, 16384, 256, 128, [17, 32, 25, 30, 64, 40, 50, 60]),
    (16, 16384, 256, 64, [18, 33] * 8),
    (6, 16384, 512, 128, [70, 96, 65, 80, 128, 90]),   # one k group per block, tiles of three row fragments
    # more blocks than CUs and larger experts: the direct-to-LDS tiles (2, 3 and 4 row fragments; 6 and 10 stages)
    (4, 16384, 768, 64, [200, 130, 75, 300]),
    (3, 16384, 1280, 128, [129, 260, 100]),
]


@pytest.mark.parametrize("E,N,K,g,rows", CASES)
def test_grouped_gemm_matches_oracle(E, N, K, g, rows):
    _say(f"grouped E={E} N={N} K={K} g={g} rows={rows}")
    ex = Experts(E, N, K, g, seed=N + K)
    ex.check(rows, seed=E, what=f"rows={rows}")


def test_grouped_equals_separate_calls_and_many_experts():
    import torch

    E, N, K, g = 64, 64, 256, 64
    _say("grouped E=64")
    ex = Experts(E, N, K, g, seed=500)
    rng = np.random.default_rng(3)
    rows = rng.integers(0, 40, size=E).tolist()
    dX, dsx, offs, ACC = ex.check(rows, seed=9, what="64 experts")
    cb, gb = api.liquidquant_packed_size(N, K, g)
    for e in (0, 17, 63):
        r0, r1 = offs[e], offs[e + 1]
        if r1 == r0:
            continue
        one = api.w4a8_gemm_i32(dX[r0:r1].contiguous(), ex.d_packed[e * cb:(e + 1) * cb],
                                ex.d_gparams[e * gb:(e + 1) * gb], N, K, g)
        torch.cuda.synchronize()
        assert torch.equal(one, ACC[r0:r1])


def test_grouped_interface_limits():
    import torch

    N, K, g = 64, 256, 64
    ex = Experts(1, N, K, g, seed=1)
    X = torch.zeros((4, K), dtype=torch.int8, device="cuda")
    sx = torch.ones(4, dtype=torch.float32, device="cuda")
    # no tokens at all: a successful no-op
    Y, _ = api.w4a8_grouped_gemm([0, 0], X[:0], sx[:0], ex.d_packed, ex.d_gparams, ex.d_w_scales, N, K, g)
    assert tuple(Y.shape) == (0, N)
    L = api.lib()
    import ctypes

    def raw(E, offs):
        arr = (ctypes.c_int * len(offs))(*offs)
        return L.w4a8_grouped_gemm(E, arr, N, K, g, ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(sx.data_ptr()),
                                   ctypes.c_void_p(ex.d_packed.data_ptr()), ctypes.c_void_p(ex.d_gparams.data_ptr()),
                                   ctypes.c_void_p(ex.d_w_scales.data_ptr()), None, None, None)

    assert raw(65, [0] * 66) == -1          # too many experts
    assert raw(0, [0]) == -1
    assert raw(1, [1, 4]) == -1             # must start at 0
    assert raw(2, [0, 3, 2]) == -1          # must not decrease
    assert raw(1, [0, 4]) == -1             # no output pointer


def test_grouped_full_size_layer_all_families():
    """A layer of realistic width (N = K = 4096, 8 experts) with experts of 5 to 700 rows, on the 16-row
    kernel and on tiles, checked in full: per expert the float64 BLAS product of the oracle's dequantised
    weights is exact (|ACC| < 2^53)."""
    import torch

    E, N, K, g = 8, 4096, 4096, 64
    rows = [5, 0, 16, 33, 64, 65, 130, 700]
    _say(f"grouped full size E={E} N={N} K={K} rows={rows}")
    Ws = [WL.make_weights(N, K, 0.02, seed=900 + e) for e in range(E)]
    packs = [api.liquidquant_pack_weights(W, g) for W in Ws]
    d_packed = torch.from_numpy(np.concatenate([p[0] for p in packs])).cuda()
    d_gparams = torch.from_numpy(np.concatenate([p[1] for p in packs])).cuda()
    d_sw = torch.from_numpy(np.stack([p[2] for p in packs])).cuda()
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(int)
    X, s_x = I.make_activations(int(offs[-1]), K, outlier_frac=0.001, seed=77)
    Y, ACC = api.w4a8_grouped_gemm(offs, torch.from_numpy(X).cuda(), torch.from_numpy(s_x).cuda(), d_packed,
                                   d_gparams, d_sw, N, K, g, want_y=True, want_acc=True)
    torch.cuda.synchronize()
    ACC, Y = ACC.cpu().numpy(), Y.cpu().numpy()
    for e in range(E):
        r0, r1 = offs[e], offs[e + 1]
        if r1 == r0:
            continue
        q = O.quantize_weights(Ws[e], g)
        assert np.array_equal(q["s_w"].view(np.uint32), packs[e][2].view(np.uint32))
        Wd = O.dequant_plain(q["Q_u4"], q["s_u8"], q["mn"], g)
        ref = X[r0:r1].astype(np.float64) @ Wd.astype(np.float64).T
        assert np.array_equal(ACC[r0:r1].astype(np.float64), ref), f"expert {e}: accumulators differ"
        H.assert_fp16_close(Y[r0:r1], ref * s_x[r0:r1, None].astype(np.float64) * q["s_w"][None, :].astype(np.float64),
                            f"expert {e}")


def _kernels(rows, N, K, g):
    """The kernels that a grouped call launches for these rows, in their order."""
    text = api.w4a8_describe_grouped([0] + [int(v) for v in np.cumsum(rows)], N, K, g)
    return [part.split("[")[0] for part in text.split("+")]


@pytest.mark.parametrize("K,kernels", [
    (1024, ["stream16_f2_w8", "solo16_pt_m256", "panel_f2_m32"]), (2304, ["stream16_f2_w8", "solo16_pt_m256", "panel_f2_m32"]),
    (768, ["stream16_f2_w8", "duo_dl_m128"])])
def test_grouped_large_experts_take_256_row_tiles(K, kernels):
    """Experts of several hundred rows on a layer wide enough that whole rounds of 256 x 256 tiles
    pay: the big experts run as one persistent launch of the one-wave-per-SIMD kernel over all of
    them (ragged last row tiles of 8, 132 and 188 rows, an expert of exactly 256 rows, tile
    boundaries between experts inside a block's stream), the small ones in their own families.
    Also with K % 512 == 256 (two added stages of zero weights per tile); with K = 768 these two are half of what
    there is, and 128-row tiles are ahead.
    Checked in full against the exact float64 product of the oracle's dequantised weights."""
    import torch

    E, N, g = 7, 4096, 128
    rows = [700, 5, 520, 900, 40, 256, 1000]
    _say(f"grouped 256-row tiles E={E} N={N} K={K} rows={rows}")
    assert _kernels(rows, N, K, g) == kernels
    Ws = [WL.make_weights(N, K, 0.02, seed=300 + e) for e in range(E)]
    packs = [api.liquidquant_pack_weights(W, g) for W in Ws]
    d_packed = torch.from_numpy(np.concatenate([p[0] for p in packs])).cuda()
    d_gparams = torch.from_numpy(np.concatenate([p[1] for p in packs])).cuda()
    d_sw = torch.from_numpy(np.stack([p[2] for p in packs])).cuda()
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(int)
    X, s_x = I.make_activations(int(offs[-1]), K, outlier_frac=0.001, seed=78)
    dX, dsx = torch.from_numpy(X).cuda(), torch.from_numpy(s_x).cuda()
    Y, ACC = api.w4a8_grouped_gemm(offs, dX, dsx, d_packed, d_gparams, d_sw, N, K, g, want_y=True, want_acc=True)
    # the accumulators alone: no scales are passed, none may be read
    _, ACC2 = api.w4a8_grouped_gemm(offs, dX, None, d_packed, d_gparams, None, N, K, g, want_y=False, want_acc=True)
    torch.cuda.synchronize()
    ACC, Y, ACC2 = ACC.cpu().numpy(), Y.cpu().numpy(), ACC2.cpu().numpy()
    assert np.array_equal(ACC, ACC2), "accumulator-only call differs"
    for e in range(E):
        r0, r1 = offs[e], offs[e + 1]
        q = O.quantize_weights(Ws[e], g)
        Wd = O.dequant_plain(q["Q_u4"], q["s_u8"], q["mn"], g)
        ref = X[r0:r1].astype(np.float64) @ Wd.astype(np.float64).T
        assert np.array_equal(ACC[r0:r1].astype(np.float64), ref), f"expert {e}: accumulators differ"
        H.assert_fp16_close(Y[r0:r1], ref * s_x[r0:r1, None].astype(np.float64) * q["s_w"][None, :].astype(np.float64),
                            f"expert {e}")


@pytest.mark.parametrize("E,N,K,g,rows", [
    (4, 320, 512, 64, [16, 17, 0, 32]),            # 32-row panels
    (3, 192, 8192, 128, [1, 9, 16]),               # ... long K: also for the smallest experts
    (3, 320, 768, 128, [33, 64, 5]),               # 64-row panels of 128 channels, a ragged last column group
    (6, 5824, 256, 64, [40, 3, 31, 17, 64, 1]),    # more blocks than one round: 32-row panels, two row tiles for some
    (6, 5824, 256, 128, [40, 33, 64, 50, 20, 1]),  # ... most experts above 32 rows: panels of both heights
    (3, 320, 512, 64, [65, 40, 20]),               # an expert of more than 64 rows: three row tiles of 32
])
def test_panel_groups(E, N, K, g, rows):
    _say(f"panel groups E={E} N={N} K={K} g={g} rows={rows}")
    Experts(E, N, K, g, seed=K).check(rows, seed=N, what=f"rows {rows}")


@pytest.mark.parametrize("N,K,g,rows,kernels", [
    # 20 row blocks: 14 on 256 x 256 tiles, 6 on 256 x 128 and a rest of 7 rows; the last tile of either kind has 64
    # channels, K % 512 == 256 adds two stages of zero weights to both
    (4416, 4864, 128, [1487, 1468, 1031, 173, 950], ["solo16_pt_m256", "solo16_g2_m256", "panel_f2_m32"]),
    (2624, 1280, 64, [1185, 949, 647], ["solo16_g2_m256"]),   # 256 x 128 tiles alone, the same edges across experts
    (3520, 4864, 64, [80, 607, 1355, 24, 636], ["solo16_g2_m256", "panel_f2_m32", "panel_f4_m64"]),   # rests on 64-row panels
    (4864, 1024, 128, [367, 29, 457, 1373], ["solo16_pt_m256", "panel_f2_m32", "panel_f4_m64"]),
    (4096, 4096, 64, [1500, 20, 1537, 1400, 1700], ["panel_f2_m32", "duo_dl_m128"]),   # rests of 1 and 120 rows in the tiles' launch
    (4096, 4864, 128, [1000, 900], ["duo_m128_g2"]),
    (4096, 4096, 64, [100, 12, 97, 128, 65], ["stream16_f2_w8", "panel_f4_m64"]),   # 64-row panels of two row tiles
    (8192, 1024, 128, [100, 97, 128, 66, 90, 100, 3, 120, 113], ["stream16_f2_w8", "duo_m128_g2"]),
    (4096, 8448, 128, [100, 12, 97, 128, 65], ["panel_f2_m32", "panel_f4_m64"]),   # long K: the smallest expert on 32-row panels
])
def test_row_blocks_and_rests(N, K, g, rows, kernels):
    """Larger experts as two kinds of 256-row tiles and what they leave over, against the float64 product
    (exact: |ACC| < 2^53) of the weights that the layout hook dequantises."""
    import torch

    _say(f"grouped row blocks N={N} K={K} g={g} rows={rows}")
    assert _kernels(rows, N, K, g) == kernels
    E = len(rows)
    cb, gb = api.liquidquant_packed_size(N, K, g)
    gen = torch.Generator(device="cuda").manual_seed(K)
    codes = torch.randint(0, 256, (cb * E,), dtype=torch.uint8, device="cuda", generator=gen)
    pairs = [torch.randint(lo, hi, (gb // 2 * E,), device="cuda", generator=gen) for lo, hi in ((1, 17), (0, 16))]
    gparams = torch.stack(pairs, 1).to(torch.uint8).reshape(-1).contiguous()   # code * s + a <= 255
    scales = torch.rand((E, N), device="cuda", generator=gen)
    offsets = [0] + [int(v) for v in np.cumsum(rows)]
    X = torch.randint(-127, 128, (offsets[-1], K), dtype=torch.int8, device="cuda", generator=gen)
    sx = torch.rand(offsets[-1], device="cuda", generator=gen) * 1e-3
    Y, ACC = api.w4a8_grouped_gemm(offsets, X, sx, codes, gparams, scales, N, K, g, want_y=True, want_acc=True)
    for e in range(E):
        lo, hi = offsets[e], offsets[e + 1]
        Wd = api.w4a8_dequant_dump(codes[e * cb:(e + 1) * cb].clone(), gparams[e * gb:(e + 1) * gb].clone(), N, K, g)
        ref = X[lo:hi].double() @ Wd.double().t()
        assert torch.equal(ACC[lo:hi].double(), ref), f"expert {e}"
        ref = ref * sx[lo:hi, None].double() * scales[e].double()
        H.assert_fp16_close(Y[lo:hi].cpu().numpy(), ref.cpu().numpy(), f"expert {e}")


@pytest.mark.parametrize("N,K,g,rows,form", [
    (4096, 4352, 64, [17, 0, 32], "panel_f1_m32"),        # 128 blocks of 64 channels, the shortest K; a last turn without units for all waves
    (4160, 4352, 64, [17, 0, 32], None),                  # 130
    (4096, 4096, 64, [17, 0, 32], None),
    (64, 14336, 128, [1, 3, 0, 16], "panel_f1_m32"),
    (1024, 4352, 128, [1, 16, 7, 2, 0, 12, 9, 3, 16], "panel_f1_m32"),   # 128 blocks of experts of up to 16 rows
    (1600, 4352, 64, [40, 66], "panel_f1_m32"),   # 125: two and three row tiles an expert, the last of one with 2 rows
])
def test_few_panels_of_long_k_take_32_channels(N, K, g, rows, form):
    text = api.w4a8_describe_grouped([0] + [int(v) for v in np.cumsum(rows)], N, K, g)
    assert text == f"panel_f2_m32[{sum(r > 0 for r in rows)} experts, {sum(rows)} rows" + (f", as {form}]" if form else "]")
    test_row_blocks_and_rests(N, K, g, rows, ["panel_f2_m32"])


@pytest.mark.parametrize("N,K,g,rows,kernels", [
    (256, 512, 64, [(37 * e) % 190 for e in range(64)], ["panel_f2_m32", "duo_m64"]),    # 52 of 64 experts in the tiles' table
    (1024, 512, 64, [65 + (37 * e) % 64 for e in range(64)], ["duo_m128_g2"]),           # the whole table
    (2048, 768, 64, [1280, 0, 1536, 1792] + [256] * 20, ["duo_dl_m128"]),
    (1024, 4096, 64, [200] * 24 + [0] * 3 + [256] * 8, ["solo16_g2_m256"]),              # ... one tile at a time
    (4096, 1024, 64, [1280, 0, 1536, 1792, 2048], ["solo16_pt_m256"]),   # row blocks in fours, the last of them 1, 2, 3 and 4
])
def test_many_experts_in_the_tiles_table(N, K, g, rows, kernels):
    test_row_blocks_and_rests(N, K, g, rows, kernels)


@pytest.mark.parametrize("E,N,K,g,rows", [
    (64, 192, 256, 64, [(7 * e) % 33 for e in range(64)]),       # the whole table: panels of up to 32 rows
    (64, 192, 512, 128, [5 + (11 * e) % 60 for e in range(64)]),  # ... 33..64 rows: one or two row tiles an expert
    (64, 2816, 256, 64, [1 + (5 * e) % 18 for e in range(64)]),   # 9.8 rounds of experts of up to 16 rows: two launches
    (2, 64, 256, 64, [17, 1]),
])
def test_many_experts_in_the_panel_table(E, N, K, g, rows):
    """Every expert against its rows as a call of its own."""
    import torch

    _say(f"panel table E={E} N={N} K={K} g={g}")
    cb, gb = api.liquidquant_packed_size(N, K, g)
    gen = torch.Generator(device="cuda").manual_seed(N)
    codes = torch.randint(0, 256, (cb * E,), dtype=torch.uint8, device="cuda", generator=gen)
    pairs = [torch.randint(lo, hi, (gb // 2 * E,), device="cuda", generator=gen) for lo, hi in ((1, 17), (0, 16))]
    gparams = torch.stack(pairs, 1).to(torch.uint8).reshape(-1).contiguous()   # code * s + a <= 255
    scales = torch.rand((E, N), device="cuda", generator=gen)
    offsets = [0] + [int(v) for v in np.cumsum(rows)]
    X = torch.randint(-127, 128, (offsets[-1], K), dtype=torch.int8, device="cuda", generator=gen)
    sx = torch.rand(offsets[-1], device="cuda", generator=gen) * 1e-3
    Y, ACC = api.w4a8_grouped_gemm(offsets, X, sx, codes, gparams, scales, N, K, g, want_y=True, want_acc=True)
    for e in range(E):
        lo, hi = offsets[e], offsets[e + 1]
        if lo == hi:
            continue
        Wd = api.w4a8_dequant_dump(codes[e * cb:(e + 1) * cb].clone(), gparams[e * gb:(e + 1) * gb].clone(), N, K, g)
        ref = X[lo:hi].cpu().numpy().astype(np.int64) @ Wd.cpu().numpy().astype(np.int64).T
        assert np.array_equal(ACC[lo:hi].cpu().numpy(), ref), f"expert {e}"
        H.assert_fp16_close(Y[lo:hi].cpu().numpy(), O.scale_epilogue_f64(ref, sx[lo:hi].cpu().numpy(), scales[e].cpu().numpy()),
                            f"expert {e}")


def test_many_small_experts_are_not_slower_together():
    """64 experts of a decode batch in one call against the same rows in two calls (up to 16 rows, more than
    16 rows).  A block that walked through the table of experts, or one launch of 32-row panels for all
    of them, took 1.4 times as long as the two calls here; 1.25 leaves room for the noise of both."""
    import torch

    E, N, K, g = 64, 2048, 1536, 64
    _say(f"many small experts E={E} N={N} K={K}")
    rows = np.random.Generator(np.random.PCG64(11)).multinomial(11 * E, [1 / E] * E)
    assert rows.max() > 16 and rows.max() <= 32
    cb, gb = api.liquidquant_packed_size(N, K, g)
    gen = torch.Generator(device="cuda").manual_seed(1)
    weights = [torch.randint(0, 256, (cb * E,), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(4)]
    gparams = torch.tensor([3, 5], dtype=torch.uint8, device="cuda").repeat(gb // 2 * E)
    scales = torch.rand((E, N), device="cuda", generator=gen)

    def calls(*parts):
        out = []
        for part in parts:
            offsets = [0] + [int(v) for v in np.cumsum(part)]
            X = torch.randint(-127, 128, (offsets[-1], K), dtype=torch.int8, device="cuda", generator=gen)
            out.append((offsets, X, torch.rand(offsets[-1], device="cuda", generator=gen)))
        return lambda i: [api.w4a8_grouped_gemm(o, X, sx, weights[i % 4], gparams, scales, N, K, g) for o, X, sx in out]

    def best_us(call, n=8):
        call(0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for i in range(n):
                call(i)
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / n)
        return min(times)

    together, apart = calls(rows), calls(np.where(rows <= 16, rows, 0), np.where(rows > 16, rows, 0))
    t, u = best_us(together), best_us(apart)
    _say(f"  one call {t:.1f} us, two calls {u:.1f} us")
    assert t < 1.25 * u
