"""16-bit products whose rows, extents or pointers are not whole 16-byte pieces, or whose C is column-major, on the matrix
cores: exact on small integers for every layout, around tile edges and K tails, against the oracle."""
import itertools

import numpy as np
import pytest
import torch

import workloads as wl
from helpers import run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


def exact(g, o, w, cfg, **kw):
    sa, sb = wl.operand_shapes(w)
    A = wl.small_integers(sa, w.seed_a, -1, 1, w.dtype)
    B = wl.small_integers(sb, w.seed_b, -1, 1, w.dtype)
    bias = wl.small_integers((w.N,), w.seed_bias, -3, 3, "f32") if w.has_bias else None
    print(f"{w.M}x{w.N}x{w.K} b{w.batch} {w.dtype} {w.layout_a}/{w.layout_b} {cfg} {kw}", flush=True)
    C, info = run_gpu(g, w, A, B, bias, config=-1 if cfg is None else g.config_names().index(cfg), return_plan_info=True, **kw)
    assert np.array_equal(wl.to_float64(C), run_oracle(o, w, A, B, bias, want=("y",))["y"]), (cfg, info)
    return info


@pytest.mark.parametrize("la,lb,lc", itertools.product(("row", "col"), ("row", "col"), ("row", "col")))
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (64, 64, 64), (65, 63, 65), (129, 255, 137), (3, 200, 191), (131, 7, 129), (257, 130, 8)])
def test_every_layout(g, oracle, la, lb, lc, M, N, K):
    """NaN-poisoned odd padding, displaced pointers, fp32 and 16-bit results."""
    for cfg in [n for n in g.config_names() if n.startswith("mfma16g_")]:
        w = wl.Workload("t", M, N, K, layout_a=la, layout_b=lb, seed_a=M + 1, seed_b=N + 2)
        exact(g, oracle, w, cfg, layout_c=lc, pad_a=3, pad_b=5, pad_c=1, out_dtype="f32")
        exact(g, oracle, wl.scaled(w, dtype="f16", epilogue="bias_relu", batch=2), cfg, layout_c=lc, pad_a=1, pad_b=1, offset_a=1, offset_b=3)


def test_built_in_choice(g, oracle):
    """Larger than the vector-ALU kernel's share, one odd extent at a time."""
    for kw in (dict(K=333), dict(N=517, layout_b="row"), dict(M=301, layout_a="col")):
        w = wl.Workload("t", **{**dict(M=304, N=520, K=336, seed_a=1, seed_b=2), **kw})
        assert "kernel=mfma16g_" in exact(g, oracle, w, None), kw


@pytest.mark.parametrize("kw,kernel", [(dict(M=613, N=21, K=15, batch=127), "general_mfma32_64x64x16"),
                                       (dict(M=2319, N=879, K=9, layout_c="col"), "general_mfma32_64x64x16"),
                                       (dict(M=697, N=41, K=37, batch=107), "mfma16g_64x64_k1_w2x2"),
                                       (dict(M=1501, N=1203, K=63, layout_a="col", layout_b="row"), "mfma16g_"),
                                       (dict(M=2463, N=1111, K=64, layout_b="row"), "mfma16g_")])
def test_built_in_choice_with_a_short_k(g, oracle, kw, kernel):
    """Up to 64 values of K, more than the vector-ALU kernel's share: one of three kernels, aligned or not."""
    lc = kw.pop("layout_c", "row")
    w = wl.Workload("t", **kw, seed_a=3, seed_b=4)
    assert "kernel=" + kernel in exact(g, oracle, w, None, layout_c=lc, out_dtype="f32")
    exact(g, oracle, w, None, layout_c=lc, pad_a=1, pad_b=3, pad_c=1, offset_a=1, offset_b=3)
