"""GPU parity at the full benchmark sizes, in the launch configuration bench.py times
(the dispatcher's own kernel choice through w4a8_gemm / w4a8_gemm_i32).

Every shape is checked two ways against the oracle's quantised weights:
  * the WHOLE accumulator matrix against the exact product X . Wd^T of the oracle's
    dequantised weights, computed with the float64 BLAS (every partial sum is an integer
    below 2^53, so the product is exact), and the WHOLE FP16 matrix against the epilogue
    definition applied to that product -- no value of the comparison comes from the GPU;
  * sampled outputs: a random set of rows x channels recomputed one by one by the oracle's
    own int64 matmul (INT32 bit-exact, FP16 within one ulp).
"""
import sys

import numpy as np
import pytest

from oracle import lqq_oracle as O
from paper_2509_01229_amd import api
from paper_2509_01229_amd import workloads as WL

import gpu_helpers as H
import inputs as I

pytestmark = pytest.mark.gpu

# 33..64 rows (panels) are not among the paper-shaped workloads: two extra batch sizes on the 7B
# up-projection cover them at full size
_M64 = [WL.GemmShape(f"mlp7b_up_M{M}_N11008_K4096", M, 11008, 4096, outlier_frac=0.001, seed=2) for M in (48, 64)]

# 33..64 rows with very long K: panels with K slices; 1280 rows on 8192 x 8192 are 160 tiles of
# 256 x 256, less than a round
_DOWN_MID = [WL.GemmShape(f"l70b_down_M{M}_N8192_K28672", M, 8192, 28672, group=128, sigma_w=0.015, seed=3)
             for M in (40, 64)]
_PREFILL_MID = [WL.GemmShape(f"prefill_M{M}_N8192_K8192", M, 8192, 8192, seed=4) for M in (56, 1280)]

FAMILIES = [
    ("decode", WL.DECODE),
    ("mlp7b_up_m64", _M64),
    ("mlp7b_up", WL.MLP_7B[:3]),
    ("mlp7b_down", WL.MLP_7B[3:]),
    ("l70b_up", WL.LAYERS_70B[0:3]),
    ("l70b_down", list(WL.LAYERS_70B[3:6]) + _DOWN_MID),
    ("l70b_qkv", WL.LAYERS_70B[6:9]),
    ("prefill", list(WL.PREFILL) + _PREFILL_MID),
]


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _oracle_exact_products(P, acts, block=2048):
    """ACC_ref[M] = X . Wd^T for every activation set, as int32: float64 BLAS on integers
    (exact: |sum| <= K * 127 * 126 < 2^53), from the oracle's quantisation in blocks of channels."""
    N = P.N
    ref = {M: np.empty((M, N), dtype=np.int32) for M in acts}
    X64 = {M: X.astype(np.float64) for M, (X, _) in acts.items()}
    s_w = np.empty(N, dtype=np.float32)
    for r0 in range(0, N, block):
        rows = np.arange(r0, min(N, r0 + block))
        Wd, s_w[rows] = P.oracle_wd(rows)
        WfT = np.ascontiguousarray(Wd.astype(np.float64).T)
        for M in acts:
            prod = X64[M] @ WfT
            assert np.abs(prod).max() < 2.0 ** 31
            ref[M][:, rows] = prod.astype(np.int32)
    return ref, s_w


@pytest.mark.parametrize("name,shapes", FAMILIES, ids=[f[0] for f in FAMILIES])
def test_full_size_family(name, shapes):
    import torch

    s0 = shapes[0]
    _say(f"{name}: generating and packing W [{s0.N} x {s0.K}] group {s0.group}")
    rng = np.random.Generator(np.random.PCG64(s0.seed))
    W = WL.make_weights(s0.N, s0.K, s0.sigma_w, rng=rng)
    P = H.Problem(s0.N, s0.K, s0.group, W=W)
    acts = {}
    for shp in shapes:
        acts[shp.M] = I.make_activations(shp.M, shp.K, shp.outlier_frac, seed=shp.seed + 1000 + shp.M)
    _say(f"{name}: exact float64 product of the oracle's weights for {sorted(acts)} rows")
    acc_ref, s_w_oracle = _oracle_exact_products(P, acts)
    assert np.array_equal(P.w_scales.view(np.uint32), s_w_oracle.view(np.uint32)), "level-1 scales differ"

    pick = np.random.default_rng(17)
    n_idx = np.sort(pick.choice(s0.N, size=192, replace=False))
    for shp in shapes:
        M = shp.M
        X, s_x = acts[M]
        vname = api.w4a8_variant_name(api.w4a8_select_variant(M, shp.N, shp.K, shp.group))
        _say(f"{shp.name}: GPU run ({vname})")
        dX, dsx = torch.from_numpy(X).cuda(), torch.from_numpy(s_x).cuda()
        Y = api.w4a8_gemm(dX, dsx, P.d_packed, P.d_gparams, P.d_w_scales, shp.N, shp.K, shp.group)
        ACC = api.w4a8_gemm_i32(dX, P.d_packed, P.d_gparams, shp.N, shp.K, shp.group)
        torch.cuda.synchronize()
        ACC = ACC.cpu().numpy()
        Y = Y.cpu().numpy()
        # every accumulator against the exact product
        assert np.array_equal(ACC, acc_ref[M]), f"{shp.name}: {np.count_nonzero(ACC != acc_ref[M])} accumulators differ"
        # sampled outputs against the oracle, element by element
        m_idx = np.arange(M) if M <= 48 else np.sort(pick.choice(M, size=48, replace=False))
        ACC_ref, Y_ref64 = P.oracle_sampled(X, s_x, m_idx, n_idx)
        assert np.array_equal(ACC[np.ix_(m_idx, n_idx)], ACC_ref), f"{shp.name}: sampled accumulators differ"
        H.assert_fp16_close(Y[np.ix_(m_idx, n_idx)], Y_ref64, shp.name)
        # whole FP16 matrix against the epilogue definition applied to the exact product
        ref64 = O.scale_epilogue_f64(acc_ref[M], s_x, s_w_oracle)
        H.assert_fp16_close(Y, ref64, shp.name + " (all outputs)")
        del ACC, Y, ref64, dX
    del P
    torch.cuda.empty_cache()
