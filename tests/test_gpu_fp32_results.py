"""fp32 results of the tiled kernels with 16-bit and fp8 operands, which leave a wave's block through LDS in pieces of 16 rows and half its
columns: exact on small integers where the last columns of C lie in either half, at either edge of one and off 16-byte pieces, where rows
end inside a piece, with rows of C at any element, in batches and on persistent workgroups that walk over several tiles."""
import pytest
import torch

import workloads as wl
from test_gpu_wide_tiles import run_exact

pytestmark = pytest.mark.gpu

NAMES = ["mfma16_256x256x64_w2x4", "mfma16_256x256x64_w2x4_p", "mfma16_256x256x64_w2x2", "mfma16_128x128x64_w2x2_s4", "mfma16t_192x256x64_w2x4",
         "mfma8_256x256x128_w2x4_s2", "mfma8_256x192x128_w4x2_s2", "mfma8_224x256x128_w2x4_s2", "mfma8_128x128x128_w2x2_s4"]


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


@pytest.mark.parametrize("cfg", NAMES)
def test_pieces_of_half_the_columns(g, cfg):
    bm, bn = (int(x) for x in cfg.split("_")[1].split("x")[:2])
    dtype = "f8" if cfg.startswith("mfma8_") else "bf16"
    strided = cfg.startswith("mfma16t_")
    kw = dict(dtype=dtype, epilogue="bias_relu", layout_b="row") if strided else dict(dtype=dtype, epilogue="bias_relu")
    for N in (1, 15, 16, 31, 32, 33, 47, 48, 49, 63, 65, 95, 97, 127, bn - 1, bn, bn + 33):
        N = -(-N // 8) * 8 if strided else N
        w = wl.Workload("t", bm - 17 if N % 2 else 33, N, 256, seed_a=N, seed_b=2, **kw)
        run_exact(g, w, cfg, out_dtype="f32", pad_c=N % 4)
    run_exact(g, wl.Workload("t", bm + 5, bn + 40, 256, batch=3, seed_a=1, seed_b=2, **kw), cfg, out_dtype="f32", pad_c=1)
    run_exact(g, wl.Workload("t", 9 * bm - 3, 40 * bn - 24, 256, seed_a=1, seed_b=2, **kw), cfg, out_dtype="f32")
