"""Launches whose tiles are walked in strips (between one and two 128x128 tiles per CU, or a K of at most 512 bytes): exact on
small integers on every kernel with such tiles, ragged last tiles, tile counts that divide by the 8 XCDs and others."""
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


@pytest.mark.parametrize("M,N,K", [(19 * 128 - 5, 15 * 128 - 8, 384), (24 * 128, 11 * 128 - 24, 320),     # 285 and 264 tiles
                                   (5 * 128 - 3, 3 * 128 - 8, 128), (17 * 128 - 40, 1280, 128), (3 * 256 - 9, 5 * 256 - 12, 256)])
def test_every_kernel_with_large_tiles(g, oracle, M, N, K):
    ran = 0
    for cfg in g.config_names():
        if not any(t in cfg for t in ("_128x128", "_256x256", "_256x192", "_256x128")) or "mfma32" in cfg or "f32mfma" in cfg:
            continue
        dtype = "f8" if cfg.startswith("mfma8_") else "bf16"
        la, lb, m, n, k = "row", "col", M, N, K
        if cfg.startswith("mfma16t_"):
            la, lb, m, n = "col", "row", M // 8 * 8, N // 8 * 8
        if cfg.startswith("mfma16g_"):
            k = K - 3
        w = wl.Workload("t", m, n, k, dtype=dtype, layout_a=la, layout_b=lb, epilogue="bias_relu", seed_a=M, seed_b=N, seed_bias=K)
        sa, sb = wl.operand_shapes(w)
        A, B = wl.small_integers(sa, w.seed_a, -1, 1, dtype), wl.small_integers(sb, w.seed_b, -1, 1, dtype)
        bias = wl.small_integers((n,), w.seed_bias, -3, 3, "f32")
        print(f"{m}x{n}x{k} {dtype} {la}/{lb} {cfg}", flush=True)
        C = run_gpu(g, w, A, B, bias, config=g.config_names().index(cfg), out_dtype="f32")
        assert np.array_equal(wl.to_float64(C), run_oracle(oracle, w, A, B, bias, want=("y",))["y"]), cfg
        ran += 1
    assert ran >= 18, ran
