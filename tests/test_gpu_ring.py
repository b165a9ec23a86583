"""The kernels with three to five slabs of K in LDS (small tiles, few rows, long K): exact on small integers around the
ring's fill and drain, K tails, tile edges, and batches whose problems are kept within an XCD."""
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


def deep_configs(g, dtype):
    family = "mfma8_" if dtype == "f8" else "mfma16_"
    return [n for n in g.config_names() if n.startswith(family) and n[-3:] in ("_s3", "_s4", "_s5")]


def exact(g, o, w, cfg, **kw):
    sa, sb = wl.operand_shapes(w)
    A = wl.small_integers(sa, w.seed_a, -1, 1, w.dtype)
    B = wl.small_integers(sb, w.seed_b, -1, 1, w.dtype)
    bias = wl.small_integers((w.N,), w.seed_bias, -3, 3, "f32") if w.has_bias else None
    print(f"{w.M}x{w.N}x{w.K} b{w.batch} {w.dtype} {cfg} {kw}", flush=True)
    C, info = run_gpu(g, w, A, B, bias, config=-1 if cfg is None else g.config_names().index(cfg), return_plan_info=True, **kw)
    assert np.array_equal(wl.to_float64(C), run_oracle(o, w, A, B, bias, want=("y",))["y"]), (cfg, info)
    return info


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f8"])
def test_every_slab_count_and_tail(g, oracle, dtype):
    """From less than one slab to several turns of the ring, with and without a tail."""
    step = 16 if dtype == "f8" else 8
    assert len(deep_configs(g, dtype)) >= 5
    for cfg in deep_configs(g, dtype):
        for K in (step, 64, 128, 192 + step, 256, 384, 512, 640 + step, 1024, 1536, 2048 + 64, 3072):
            exact(g, oracle, wl.Workload("t", 33, 47, K, dtype=dtype, seed_a=K, seed_b=K + 1), cfg, out_dtype="f32")


@pytest.mark.parametrize("dtype", ["bf16", "f8"])
@pytest.mark.parametrize("M,N,batch", [(17, 31, 1), (64, 64, 1), (65, 129, 1), (130, 260, 1), (40, 72, 8), (129, 130, 2), (100, 64, 5)])
def test_tile_edges_and_batches(g, oracle, dtype, M, N, batch):
    """Ragged tiles in both directions; batches of a multiple of 8 tiles (whole problems per XCD) and others."""
    for cfg in deep_configs(g, dtype):
        # |sum| <= K + 3 = 211 < 256: every result is exact in bf16
        w = wl.Workload("t", M, N, 208, dtype=dtype, out_dtype="bf16", batch=batch, epilogue="bias_relu", seed_a=M, seed_b=N + 1)
        exact(g, oracle, w, cfg)
        exact(g, oracle, w, cfg, pad_a=16, pad_b=16, pad_c=1)        # C rows that are not 8-byte aligned


def test_built_in_choice(g, oracle):
    """Few rows, few tiles, long K."""
    for dtype, M, N, K in (("bf16", 64, 1024, 4096), ("f16", 200, 300, 2048), ("f8", 32, 2048, 4096)):
        info = exact(g, oracle, wl.Workload("t", M, N, K, dtype=dtype, seed_a=1, seed_b=2), None, out_dtype="f32")
        assert any(s in info for s in ("_s3 ", "_s4 ", "_s5 ")), info
