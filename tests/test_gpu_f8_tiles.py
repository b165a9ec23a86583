"""The tiled fp8 kernels (16x16x128 instruction): exact on small integers around the hand-over of the first and last slabs, K tails,
ragged tiles, C rows at any element, batches, and persistent workgroups that walk over several tiles."""
import pytest
import torch

import workloads as wl
from test_gpu_wide_tiles import run_exact

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


CONFIGS = ["mfma8_256x256x128_w2x4_s2", "mfma8_224x256x128_w2x4_s2", "mfma8_192x256x128_w2x4_s2", "mfma8_256x192x128_w4x2_s2",
           "mfma8_128x128x128_w2x2_s2", "mfma8_128x128x128_w2x2_s4"]


@pytest.mark.parametrize("cfg", CONFIGS)
def test_slabs_tails_edges_and_batches(g, cfg):
    """Persistent workgroups where K is two or more whole slabs of 128 (the _s2 configurations), one tile per workgroup otherwise.
    (|sum| <= 656 + 3: exact in fp32 output; bf16 output is the same rounding of the same value.)"""
    bm, bn = (int(x) for x in cfg.split("_")[1].split("x")[:2])
    for M, N, K in [(bm, bn, 256), (bm - 8, bn + 8, 384), (bm + 8, bn - 8, 512), (8, 8, 640), (2 * bm + 16, bn + 8, 640), (bm, bn, 128),
                    (bm + 32, 40, 16), (bm - 24, bn, 144), (bm + 8, bn, 400), (200, 264, 656), (24, 264, 112)]:
        w = wl.Workload("t", M, N, K, dtype="f8", out_dtype="bf16", epilogue="bias_relu", seed_a=K, seed_b=M)
        run_exact(g, w, cfg, out_dtype="f32")
        run_exact(g, w, cfg)
    for K in (256, 272):
        w = wl.Workload("t", bm + 8, bn + 3, K, dtype="f8", out_dtype="bf16", epilogue="bias_relu", seed_a=2, seed_b=3)
        run_exact(g, w, cfg, pad_c=3)
        run_exact(g, w, cfg, pad_c=1, out_dtype="f32")
        run_exact(g, wl.Workload("t", bm + 8, bn + 8, K, dtype="f8", out_dtype="bf16", batch=3, seed_a=1, seed_b=2), cfg, out_dtype="f32")
    for M, N, K, batch in ((3000, 6000, 256, 1), (2304, 8192, 384, 1), (504, 1000, 256, 41)):   # more tiles than CUs, also a batch
        run_exact(g, wl.Workload("t", M, N, K, dtype="f8", out_dtype="bf16", batch=batch, seed_a=K, seed_b=N), cfg)


@pytest.mark.parametrize("cfg", ["mfma8_256x256x128_w2x4_one", "mfma8_224x256x128_w2x4_one", "mfma8_192x256x128_w2x4_one", "mfma8_256x192x128_w4x2_one",
                                 "mfma8_128x128x128_w2x2_one"])
def test_one_tile_per_workgroup_whatever_k_is(g, cfg):
    test_slabs_tails_edges_and_batches(g, cfg)
