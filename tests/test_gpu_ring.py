"""The kernels with three to five slabs of K in LDS (small tiles, few rows, long K): exact on small integers around the
ring's fill and drain, K tails, tile edges, and batches whose problems are kept within an XCD."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import gpu_desc, run_gpu, run_oracle

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


@pytest.mark.parametrize("K", [328, 384])                    # with a K tail: 328 = 2 x 128 + 72 = 256 + 72 = 5 x 64 + 8 = 10 x 32 + 8
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_special_values_as_on_the_general_kernel(g, dtype, K):
    """Subnormal, infinite and NaN operands and products that overflow, in whole slabs and in the K tail, beside ragged
    tile edges: the same values as from the general kernel, which multiplies in fp32, and none of them in another row or
    column.  The deep kernels and those for any alignment in every layout they take; fp32 the kernels with slabs in LDS."""
    M, N = 72, 136
    dt = wl.TORCH_DTYPE[dtype]
    v = [torch.finfo(dt).smallest_normal / 4, -torch.finfo(dt).smallest_normal / 2, float("inf"), float("nan"),
         torch.finfo(dt).max, 1.0, -float("inf")]
    A, B = torch.zeros((1, M, K), dtype=dt), torch.zeros((1, N, K), dtype=dt)
    for i, x in enumerate(v):
        for k in (i, 250 + i, K - 1 - i):                    # a special value per row; rows differ in where it is
            A[0, 7 * (k % 10) + i:7 * (k % 10) + i + 1, k] = x
            B[0, :, k] = torch.tensor([1.0, 2.0, -0.0, 4.0], dtype=dt).repeat(N // 4)
    B[0, 5, 3] = float("inf")                                # one column of C: infinity times zero
    B[0, 131, K - 2] = float("nan")
    general = g.config_names().index("general_mfma32_64x64x16")
    wanted = ("f32mfma_",) if dtype == "f32" else ("mfma16_", "mfma16t_", "mfma16g_")
    seen = set()
    for la in ("row", "col"):
        for lb in ("col", "row"):
            Al = A if la == "row" else A.transpose(1, 2).contiguous()
            Bl = B if lb == "col" else B.transpose(1, 2).contiguous()
            w = wl.Workload("t", M, N, K, dtype=dtype, layout_a=la, layout_b=lb)
            want = run_gpu(g, w, Al, Bl, None, out_dtype="f32", config=general)
            assert 0 < int(torch.isnan(want).sum()) < want.numel() // 4 and bool(torch.isinf(want).any())
            for i, n in enumerate(g.config_names()):
                if not n.startswith(wanted):
                    continue
                pad = 1 if n.startswith("mfma16g_") else 0   # (that kernel takes what is not whole 16-byte pieces)
                try:
                    g.gemm_destroy(g.gemm_create_config(gpu_desc(g, w, "f32", lda=Al.shape[2] + pad, ldb=Bl.shape[2] + pad), i))
                except g.GemmError:
                    continue                                  # another layout's kernel
                print(f"{dtype} {la}/{lb} {n}", flush=True)
                got = run_gpu(g, w, Al, Bl, None, out_dtype="f32", config=i, pad_a=pad, pad_b=pad)
                assert torch.equal(torch.isnan(got), torch.isnan(want)), n
                assert torch.equal(torch.nan_to_num(got, nan=0.5), torch.nan_to_num(want, nan=0.5)), n
                seen.add((la, lb, n))
    assert len(seen) >= (8 if dtype == "f32" else 25), seen
