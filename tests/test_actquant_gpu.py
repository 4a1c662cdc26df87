"""GPU parity of the per-token activation quantisation kernel (Sec. 6 of the paper) against
the CPU oracle: INT8 codes and FP32 scales must match bit for bit (every step is one
correctly rounded FP32 operation on both sides), and the chain quantise -> W4A8 GEMM must
reproduce the oracle chain."""
import sys

import numpy as np
import pytest

from oracle import lqq_oracle as O
from paper_2509_01229_amd import api
from paper_2509_01229_amd import workloads as WL

import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _run(X16, smooth):
    import torch

    dX = torch.from_numpy(X16).cuda()
    ds = torch.from_numpy(smooth).cuda() if smooth is not None else None
    q, s = api.w4a8_quantize_activations(dX, ds)
    torch.cuda.synchronize()
    return q.cpu().numpy(), s.cpu().numpy()


SHAPES = [
    (1, 8), (1, 256), (7, 4096), (33, 11008), (16, 8192), (3, 16384),  # register-resident tokens
    (2, 16392), (5, 28672), (3, 32768),                               # register-resident on 1024 threads, ragged tail
    (2, 32776), (2, 131072),                                          # two-pass tokens
    (300, 512),                                                       # many short tokens
]


@pytest.mark.parametrize("M,K", SHAPES)
@pytest.mark.parametrize("with_smooth", [False, True])
def test_quantize_activations_bit_exact(M, K, with_smooth):
    _say(f"actquant M={M} K={K} smooth={with_smooth}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=M + K)
    smooth = WL.make_smooth(K, seed=K) if with_smooth else None
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


@pytest.mark.parametrize("M,K", [(1027, 2048), (2051, 4096), (4096, 512), (1027, 12288), (600, 16384)])
def test_several_tokens_per_block(M, K):
    """From 1024 tokens of 2049 to 16384 columns on a block quantises several consecutive tokens (here 5,
    with a ragged last block) and shares the reciprocals of the smooth scales between them: the second and
    fourth case.  The others were such cases once and are blocks of one token."""
    _say(f"actquant rows per block M={M} K={K}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=M)
    smooth = WL.make_smooth(K, seed=K + 1)
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


# the block shapes change at these columns (pieces of 8 per thread and threads per token) and with 1024
# tokens (several per block)
@pytest.mark.parametrize("K", [2040, 2056, 4096, 4104, 8192, 8200, 12296, 16384, 16392, 32768])
@pytest.mark.parametrize("M", [1, 32, 43, 65, 513])
@pytest.mark.parametrize("with_smooth", [False, True])
def test_edges_of_the_block_shapes(M, K, with_smooth):
    _say(f"actquant block shapes M={M} K={K} smooth={with_smooth}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=M * 7 + K)
    smooth = WL.make_smooth(K, seed=K + 2) if with_smooth else None
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


# four blocks share a token up to 64 tokens, two up to 128 (in grids padded to 8 tokens); 768 threads from 4104 to
# 6144 and from 8200 to 12288 columns, 1024 threads of two pieces up to 16384; the outlier channels put most
# values of a token near few integers, the values +-k/2 of the first columns on and next to ties of scale 1
@pytest.mark.parametrize("K", [4104, 6144, 6152, 8200, 12288, 16384, 28680])
@pytest.mark.parametrize("M", [9, 64, 65, 128, 129, 512])
@pytest.mark.parametrize("with_smooth", [False, True])
def test_edges_of_shared_tokens(M, K, with_smooth):
    _say(f"actquant shared tokens M={M} K={K} smooth={with_smooth}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=M * 3 + K)
    ties = (np.arange(1024) % 255 - 127).astype(np.float16) / 2
    X16[:, :1024] = ties
    X16[0::2, 1] = 127.0
    smooth = np.ones(K, dtype=np.float32) if with_smooth else None
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


@pytest.mark.parametrize("M,K", [(1023, 2056), (1024, 2056), (1025, 4104), (1537, 8200), (1024, 8192), (1025, 16384), (1030, 12296)])
def test_edges_of_several_tokens_per_block(M, K):
    """Odd and even numbers of tokens per block, ragged last blocks and ragged last pieces."""
    _say(f"actquant several tokens M={M} K={K}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=M + 1)
    smooth = WL.make_smooth(K, seed=K + 3)
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


@pytest.mark.parametrize("M,K", [(1023, 4104), (1024, 4104), (1025, 6144), (2047, 6152), (2048, 6152), (2049, 8192), (2048, 8200)])
def test_edges_of_many_tokens_without_smooth_scales(M, K):
    _say(f"actquant many tokens M={M} K={K}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=M + 2)
    q_ref, s_ref = O.quantize_activations(X16, None)
    q, s = _run(X16, None)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


@pytest.mark.parametrize("M,K", [(6200, 16384), (8192, 12296)])
def test_large_calls_equal_their_parts(M, K):
    """From 96 M elements on fewer blocks share a CU (without smooth scales, 12289 to 16384 columns)."""
    import torch

    _say(f"actquant large call M={M} K={K}")
    X = torch.randn((M, K), device="cuda").half()
    q, s = api.w4a8_quantize_activations(X)
    for lo, hi in ((0, M // 2), (M // 2, M)):
        qp, sp = api.w4a8_quantize_activations(X[lo:hi].clone())
        assert torch.equal(q[lo:hi], qp) and torch.equal(s[lo:hi], sp)


def test_a_few_columns_more_do_not_cost_a_larger_block():
    """8192 tokens of 4104 columns against 4096: blocks with twice the threads for one piece more took 1.37
    times as long; 1.2 leaves room for the noise of both."""
    import torch

    def best_us(K):
        X = [torch.randn((8192, K), device="cuda").half() for _ in range(6)]   # (beyond the caches)
        api.w4a8_quantize_activations(X[0])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for x in X:
                api.w4a8_quantize_activations(x)
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / len(X))
        return min(times)

    t, u = best_us(4104), best_us(4096)
    _say(f"actquant 8192 x 4104 {t:.1f} us, 8192 x 4096 {u:.1f} us")
    assert t < 1.2 * u


# (up to 1023 tokens every division is the IEEE one; the other shapes are the three block shapes of several tokens,
# which take the short division where all scales of a thread are in range)
@pytest.mark.parametrize("M,K", [(5, 2048), (1025, 2056), (1025, 8192), (1030, 12296)])
def test_smooth_scales_outside_the_short_division_range(M, K):
    """Smooth scales below 2^-40 or above 2^40 (and FP32 subnormals) take the full IEEE
    division; scales at the edges of the range and powers of two take the short one."""
    _say(f"actquant extreme smooth scales M={M} K={K}")
    rng = np.random.default_rng(5)
    X16 = (rng.standard_normal((M, K)) * 3).astype(np.float16)
    X16[1] = (rng.standard_normal(K) * 1e-4).astype(np.float16)       # FP16 subnormals among them
    X16[2, ::3] = np.float16(65504.0)
    smooth = np.exp2(rng.integers(-45, 46, size=K)).astype(np.float32)   # in and out of range within a thread's columns
    smooth[::7] *= np.float32(1.2345)
    smooth[K // 2:] = np.exp2(rng.uniform(-40, 40, size=K - K // 2))     # ... and whole threads in range
    smooth[3] = smooth[K - 3] = np.float32(2.0 ** -40)
    smooth[4] = smooth[K - 4] = np.float32(2.0 ** 40)
    smooth[5] = np.float32(1e-38)      # the quotients overflow or are huge: codes saturate
    smooth[6] = np.float32(1e-44)      # FP32 subnormal
    X16[:-2, 5:7] = 0                  # all but the last two tokens stay finite; those overflow (unspecified codes)
    X16[-2:, 5:7] = 1
    with np.errstate(over="ignore", invalid="ignore"):
        q_ref, s_ref = O.quantize_activations(X16, smooth)
    finite = np.isfinite(s_ref)
    assert finite[:-2].all() and not finite[-2:].any()
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32)[finite], s_ref.view(np.uint32)[finite])
    assert np.array_equal(q[finite], q_ref[finite])
    assert np.isinf(s[~finite]).all()
    # and a moderate range, where every token stays finite and every thread may take the short division
    smooth = np.exp2(rng.uniform(-12, 12, size=K)).astype(np.float32)
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    q, s = _run(X16, smooth)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(q, q_ref)


def test_infinite_activations_do_not_depend_on_the_batch():
    """A token's scale is that of the definition, x / smooth in FP32, however many tokens share the call:
    infinite where an activation is, and unmoved by the NaN of another channel (the codes of such
    tokens are unspecified)."""
    import torch

    _say("actquant infinite activations")
    for K in (2056, 8192, 12296):
        X16 = WL.make_activations_f16(1031, K, seed=K)
        X16[3, 5], X16[500, K - 1], X16[1030, 0], X16[7, 9] = np.inf, -np.inf, np.inf, np.nan
        smooth = WL.make_smooth(K, seed=K + 4)
        q, s = _run(X16, smooth)
        some = [0, 3, 7, 8, 500, 1029, 1030]
        q_few, s_few = _run(X16[some], smooth)
        assert np.isinf(s[[3, 500, 1030]]).all() and np.isfinite(np.delete(s, [3, 500, 1030])).all()
        assert np.array_equal(s[some], s_few) and np.array_equal(q[some], q_few)
        x = X16.copy()
        x[[3, 500, 1030, 7]] = 0
        q_ref, s_ref = O.quantize_activations(x, smooth)
        keep = np.delete(np.arange(1031), [3, 7, 500, 1030])
        assert np.array_equal(s[keep], s_ref[keep]) and np.array_equal(q[keep], q_ref[keep])


def test_quantize_activations_edge_values():
    _say("actquant edge values")
    K = 512
    X = np.zeros((6, K), dtype=np.float16)
    X[1, 5] = 65504.0                       # largest FP16
    X[1, 6] = -65504.0
    X[1, 7] = 257.9                         # rounds to a small code
    X[2, :] = 6e-8                          # FP16 subnormals only
    X[3, :] = np.float16(-1.0)              # constant token
    X[4, ::2] = 0.5
    X[4, 1::2] = 1.0                        # exact ties: 0.5 / (1/127) = 63.5 -> 64
    X[5, 3] = 1.0                           # one-hot
    q_ref, s_ref = O.quantize_activations(X)
    q, s = _run(X, None)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(q, q_ref)
    assert s[0] == 1.0 and not q[0].any()
    assert q[1, 5] == 127 and q[1, 6] == -127 and q[3].tolist() == [-127] * K
    assert q[4, 0] == 64 and q[4, 1] == 127


def test_quantize_activations_near_ties():
    """Tokens whose quotients sit on or next to rounding ties: x = k/2 * s for all k, and the
    FP16 neighbours of those values."""
    _say("actquant near ties")
    K = 512
    rows = []
    for amax in (1.0, 127.0, 0.3333, 100.0):
        base = (np.arange(K) % 255 - 127).astype(np.float64) * 0.5 * (amax / 127.0)
        for bump in (0, 1, -1):
            x = base.astype(np.float16)
            x = (x.view(np.int16) + np.int16(bump)).view(np.float16) if bump else x
            x[0] = amax
            rows.append(np.nan_to_num(x, nan=0.0, posinf=0.0, neginf=0.0))
    X = np.stack(rows).astype(np.float16)
    for smooth in (None, WL.make_smooth(K, seed=3)):
        q_ref, s_ref = O.quantize_activations(X, smooth)
        q, s = _run(X, smooth)
        assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32))
        assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


@pytest.mark.parametrize("with_smooth", [False, True])
def test_more_tokens_than_a_launch_takes(with_smooth):
    """2^24 tokens of one block of 256 threads each would be 2^32 threads: several launches, with the
    results of calls of their own."""
    import torch

    M, K = (1 << 24) + 5, 8
    _say(f"actquant M={M} K={K} smooth={with_smooth}")
    X = torch.randn((M, K), device="cuda").half()
    smooth = torch.from_numpy(WL.make_smooth(K, seed=K)).cuda() if with_smooth else None
    q, s = api.w4a8_quantize_activations(X, smooth)
    for lo, hi in ((0, 70), ((1 << 21) - 3, (1 << 21) + 5), ((1 << 23) - 3, (1 << 23) + 5), (M - 70, M)):
        qp, sp = api.w4a8_quantize_activations(X[lo:hi].clone(), smooth)
        assert torch.equal(q[lo:hi], qp) and torch.equal(s[lo:hi], sp)


def test_empty_and_bad_arguments():
    import torch

    X0 = torch.empty((0, 256), dtype=torch.float16, device="cuda")
    q, s = api.w4a8_quantize_activations(X0)
    assert tuple(q.shape) == (0, 256) and tuple(s.shape) == (0,)
    with pytest.raises(api.LiquidGemmError):
        api.w4a8_quantize_activations(torch.zeros((2, 12), dtype=torch.float16, device="cuda"))
    with pytest.raises(TypeError):
        api.w4a8_quantize_activations(torch.zeros((2, 16), dtype=torch.float32, device="cuda"))
    with pytest.raises(ValueError):
        api.w4a8_quantize_activations(torch.zeros((2, 16), dtype=torch.float16, device="cuda"),
                                      torch.ones(8, dtype=torch.float32, device="cuda"))


def test_quantize_then_gemm_matches_oracle_chain():
    import torch

    M, N, K, g = 24, 256, 1024, 64
    _say("actquant -> gemm chain")
    P = H.Problem(N, K, g, seed=21)
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.002, seed=22)
    smooth = WL.make_smooth(K, seed=23)
    q_ref, s_ref = O.quantize_activations(X16, smooth)
    ACC_ref, _ = P.oracle_gemm(q_ref, s_ref)
    ref64 = O.scale_epilogue_f64(ACC_ref, s_ref, P.oracle_full()["s_w"])
    dq, ds = api.w4a8_quantize_activations(torch.from_numpy(X16).cuda(), torch.from_numpy(smooth).cuda())
    Y = api.w4a8_gemm(dq, ds, P.d_packed, P.d_gparams, P.d_w_scales, N, K, g)
    ACC = api.w4a8_gemm_i32(dq, P.d_packed, P.d_gparams, N, K, g)
    torch.cuda.synchronize()
    assert np.array_equal(ACC.cpu().numpy(), ACC_ref)
    H.assert_fp16_close(Y.cpu().numpy(), ref64, "chain")


def _us(X16s, n=24, reps=9):
    """Microseconds a call, from replays of a graph that takes the inputs in turn (the median replay)."""
    import torch

    outs = [(torch.empty(x.shape, dtype=torch.int8, device="cuda"), torch.empty(x.shape[0], device="cuda")) for x in X16s]

    def calls():
        for i in range(n):
            api.w4a8_quantize_activations(X16s[i % len(X16s)], out_q=outs[i % len(X16s)][0], out_scales=outs[i % len(X16s)][1])

    calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    times = []
    for _ in range(reps + 1):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / n)
    return sorted(times[1:])[reps // 2]


@pytest.mark.parametrize("M,K", [(2854, 6264), (1311, 27584)])
def test_tokens_full_of_ties_are_not_much_slower(M, K):
    """Every value half an integer of scale 1, so that each needs the division.  A loop over a lane's ties, one selected at
    a time, took 2.7 times as long as on Gaussian values; the divisions one by one or all 8 take 1.5 to 1.7 times."""
    import torch

    _say(f"actquant ties M={M} K={K}")
    gen = torch.Generator(device="cuda").manual_seed(K)
    gauss = [torch.randn((M, K), device="cuda", generator=gen).half() for _ in range(4)]
    ties = [torch.randint(-126, 126, (M, K), device="cuda", generator=gen).half() + 0.5 for _ in range(4)]
    for x in ties:
        x[:, 0] = 127
    q, s = api.w4a8_quantize_activations(ties[0])
    assert torch.equal(s, torch.ones_like(s)) and torch.equal(q, torch.round(ties[0].float()).to(torch.int8))
    g, t = _us(gauss), _us(ties)
    _say(f"  Gaussian {g:.1f} us, ties {t:.1f} us")
    assert t < 2.1 * g


@pytest.mark.parametrize("M,K", [(2047, 8200), (2048, 8200), (2049, 10240), (2048, 10248), (2050, 9000)])
def test_edges_of_three_pieces(M, K):
    """512 threads of three pieces from 2048 tokens and 8200 to 10240 columns, 768 of two around that."""
    _say(f"actquant three pieces M={M} K={K}")
    X16 = WL.make_activations_f16(M, K, outlier_frac=0.001, seed=K)
    X16[:, :1024] = (np.arange(1024) % 255 - 127).astype(np.float16) / 2
    X16[0::2, 1] = 127.0
    q_ref, s_ref = O.quantize_activations(X16, None)
    q, s = _run(X16, None)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32)), "per-token scales differ"
    assert np.array_equal(q, q_ref), f"{np.count_nonzero(q != q_ref)} codes differ"


def test_block_shape_past_8192_columns():
    """Many tokens of 8680 columns keep the pace of 8192.  768 threads of two pieces, nearly a third of them past the
    end, took 1.05 to 1.11 of the time of 512 threads of three there."""
    import torch

    _say("actquant 7880 tokens of 8192 and 8680 columns")
    gen = torch.Generator(device="cuda").manual_seed(1)
    a, b = ([torch.randn((7880, K), device="cuda", generator=gen).half() for _ in range(4)] for K in (8192, 8680))
    t, u = (min(v) for v in zip(*((_us(a) / 8192, _us(b) / 8680) for _ in range(4))))   # (in turn: the clocks drift)
    _say(f"  {7880 * 3e-6 / t:.2f} and {7880 * 3e-6 / u:.2f} TB/s")
    assert u < 1.025 * t
