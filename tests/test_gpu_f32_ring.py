"""fp32 products with slabs of K straight to LDS: bit exact on small integers for every layout, around tile edges, K tails
and the ring's fill and drain, for both tile sizes."""
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


@pytest.mark.parametrize("la,lb", [("row", "row"), ("row", "col"), ("col", "row"), ("col", "col")])
@pytest.mark.parametrize("M,N,K,batch", [(4, 4, 4, 1), (64, 64, 32, 1), (68, 132, 36, 1), (128, 64, 64, 8), (132, 260, 100, 3), (260, 72, 128, 2), (192, 128, 292, 1)])
def test_exact(g, oracle, la, lb, M, N, K, batch):
    for cfg in ("f32mfma_64x64x32", "f32mfma_128x128x32"):
        for lc in ("row", "col"):
            w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, batch=batch, epilogue="bias_relu",
                            seed_a=M + 1, seed_b=N + 2)
            sa, sb = wl.operand_shapes(w)
            A = wl.small_integers(sa, w.seed_a, -2, 2, "f32")
            B = wl.small_integers(sb, w.seed_b, -2, 2, "f32")
            bias = wl.small_integers((N,), w.seed_bias, -3, 3, "f32")
            print(f"{M}x{N}x{K} b{batch} {la}/{lb}/{lc} {cfg}", flush=True)
            C = run_gpu(g, w, A, B, bias, config=g.config_names().index(cfg), layout_c=lc, pad_a=4, pad_b=8, pad_c=1)
            assert np.array_equal(wl.to_float64(C), run_oracle(oracle, w, A, B, bias, want=("y",))["y"]), (cfg, lc)


@pytest.mark.parametrize("la,lb", [("row", "row"), ("row", "col"), ("col", "row"), ("col", "col")])
@pytest.mark.parametrize("huge", ["a", "b"])
def test_leading_dimensions_beyond_32_bit_offsets(g, oracle, la, lb, huge):
    """A leading dimension of 2^24 elements: a tile's rows do not fit 32-bit offsets and the plans run the kernel that stages
    its slabs through registers (both tile sizes, every layout pair; 2.4 to 4.9 GB of address space, few rows touched)."""
    M, N, K, ld = 72, 68, 36, 1 << 24
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, epilogue="bias_relu", seed_a=1, seed_b=2)
    sa, sb = wl.operand_shapes(w)
    A, B = wl.small_integers(sa, w.seed_a, -2, 2, "f32"), wl.small_integers(sb, w.seed_b, -2, 2, "f32")
    bias = wl.small_integers((N,), w.seed_bias, -3, 3, "f32")
    dev = torch.device("cuda:0")
    Ad, Bd, biasd = A.to(dev), B.to(dev), bias.to(dev)
    src = Ad if huge == "a" else Bd
    wide = torch.empty(((src.shape[1] - 1) * ld + src.shape[2],), dtype=torch.float32, device=dev)
    rows = wide.as_strided((src.shape[1], src.shape[2]), (ld, 1))
    rows.copy_(src[0])
    want = run_oracle(oracle, w, A, B, bias, want=("y",))["y"]
    for cfg in ("f32mfma_64x64x32", "f32mfma_128x128x32"):
        C = torch.full((1, M, N), -777.0, device=dev)
        lds = {"lda": ld} if huge == "a" else {"ldb": ld}
        plan = g.gemm_create_config(gpu_desc(g, w, **lds), g.config_names().index(cfg))
        print(f"{la}/{lb} {huge} {plan.info()}", flush=True)
        g.gemm_run(plan, rows if huge == "a" else Ad, rows if huge == "b" else Bd, C, biasd)
        torch.cuda.synchronize()
        g.gemm_destroy(plan)
        assert np.array_equal(wl.to_float64(C.cpu()), want), cfg


@pytest.mark.parametrize("la,lb,lc", [("row", "row", "row"), ("row", "col", "col"), ("col", "row", "row"), ("col", "col", "row")])
@pytest.mark.parametrize("M,N,K,batch", [(828, 4100, 4, 1), (828, 4100, 36, 1), (124, 188, 192, 150), (828, 4100, 196, 1)])
def test_built_in_choice_around_the_short_k_rule(g, oracle, la, lb, lc, M, N, K, batch):
    """Three to four 64x64 tiles per CU: the staged kernel up to K = 192, slabs straight to LDS above; displaced operands run the
    general kernel on either plan's grid."""
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, batch=batch, epilogue="bias_relu", seed_a=M, seed_b=N)
    sa, sb = wl.operand_shapes(w)
    A, B = wl.small_integers(sa, w.seed_a, -2, 2, "f32"), wl.small_integers(sb, w.seed_b, -2, 2, "f32")
    bias = wl.small_integers((N,), w.seed_bias, -3, 3, "f32")
    want = run_oracle(oracle, w, A, B, bias, want=("y",))["y"]
    for kw in (dict(pad_a=4, pad_c=1), dict(offset_a=1), dict(offset_b=3)):
        print(f"{M}x{N}x{K} b{batch} {la}/{lb}/{lc} {kw}", flush=True)
        C, info = run_gpu(g, w, A, B, bias, layout_c=lc, return_plan_info=True, **kw)
        assert "kernel=f32mfma_64x64x32" in info and (int(info.split(" lds=")[1].split()[0]) == 49152) == (K > 192), info
        assert np.array_equal(wl.to_float64(C), want), (kw, info)
