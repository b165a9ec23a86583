"""16-bit products whose operands are not K-contiguous (a plain row-major product, a layer's backward pass) on the
tiled matrix-core kernels: exact on small integers at the edges of tiles, slabs and K tails, for every layout pair."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import assert_parity, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

PAIRS = [("row", "row"), ("col", "row"), ("col", "col")]


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


def configs(g, persistent):
    return [n for n in g.config_names() if n.startswith("mfma16t_") and n.endswith("_p") == persistent]


def exact(g, o, w, cfg, out_dtype=None, **kw):
    sa, sb = wl.operand_shapes(w)
    A = wl.small_integers(sa, w.seed_a, -1, 1, w.dtype)
    B = wl.small_integers(sb, w.seed_b, -1, 1, w.dtype)
    bias = wl.small_integers((w.N,), w.seed_bias, -3, 3, "f32") if w.has_bias else None
    print(f"{w.M}x{w.N}x{w.K} b{w.batch} {w.dtype} {w.layout_a}/{w.layout_b} {cfg} {kw}", flush=True)
    C, info = run_gpu(g, w, A, B, bias, config=-1 if cfg is None else g.config_names().index(cfg), out_dtype=out_dtype,
                      return_plan_info=True, **kw)
    assert np.array_equal(wl.to_float64(C), run_oracle(o, w, A, B, bias, want=("y",))["y"]), (cfg, info)
    return info


@pytest.mark.parametrize("la,lb", PAIRS)
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (256, 256, 64), (264, 520, 200), (136, 120, 72), (248, 776, 640), (520, 264, 1)])
def test_one_tile_per_workgroup(g, oracle, la, lb, M, N, K):
    """Ragged last tiles, K tails, one to ten slabs; K any where neither operand is K-contiguous."""
    if "row" == la or lb == "col":
        K = max(8, K // 8 * 8)
    else:
        K = K + 3 if K > 8 else K
    for cfg in configs(g, False):
        exact(g, oracle, wl.Workload("t", M, N, K, layout_a=la, layout_b=lb, seed_a=M + 1, seed_b=N + 2), cfg)
        exact(g, oracle, wl.Workload("t", M, N, K, dtype="f16", layout_a=la, layout_b=lb, seed_a=M + 3, seed_b=N + 4,
                                     epilogue="bias_relu"), cfg, out_dtype="f32", pad_a=8, pad_b=16, pad_c=3)


@pytest.mark.parametrize("la,lb", PAIRS)
@pytest.mark.parametrize("M,N,K,batch", [(256, 256, 128, 1), (264, 520, 192, 1), (1032, 264, 320, 3), (392, 264, 128, 64)])
def test_persistent_workgroups(g, oracle, la, lb, M, N, K, batch):
    """Two slabs and more, batches, several tiles per workgroup (the last case: 768 tiles of 128 x 128)."""
    for cfg in configs(g, True):
        w = wl.Workload("t", M, N, K, layout_a=la, layout_b=lb, batch=batch, seed_a=M + 1, seed_b=N + 2)
        exact(g, oracle, w, cfg, pad_a=8)
        exact(g, oracle, w, cfg, out_dtype="f32", pad_c=1)       # C rows that start at any element


@pytest.mark.parametrize("la,lb", PAIRS)
def test_built_in_choice_and_unaligned_pointers(g, oracle, la, lb):
    """The built-in choice takes these kernels; pointers that are only element-aligned run the general kernel."""
    w = wl.Workload("t", 776, 1032, 456, layout_a=la, layout_b=lb, seed_a=1, seed_b=2)
    assert "kernel=mfma16t_" in exact(g, oracle, w, None)
    exact(g, oracle, w, None, offset_a=1)
    exact(g, oracle, w, None, offset_b=3)
    sa, sb = wl.operand_shapes(w)
    A, B = wl._draw(("normal", 1.0), sa, 5).to(torch.bfloat16), wl._draw(("normal", 0.05), sb, 6).to(torch.bfloat16)
    C = run_gpu(g, w, A, B, None, out_dtype="f32")
    assert_parity(w, C, run_oracle(oracle, w, A, B, None), A, B, None, out_dtype="f32")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_special_values_as_on_the_general_kernel(g, dtype):
    """Subnormal, infinite and NaN operands, and sums that overflow: the same values (all exact or special) from the
    tiled kernels as from the general one, which multiplies in fp32."""
    M, N, K = 136, 264, 72
    w = wl.Workload("t", M, N, K, dtype=dtype, layout_a="col", layout_b="row")
    dt = wl.TORCH_DTYPE[dtype]
    A, B = torch.zeros((1, K, M), dtype=dt), torch.zeros((1, K, N), dtype=dt)
    tiny = torch.finfo(dt).smallest_normal
    for i, v in enumerate([tiny / 4, -tiny / 2, float("inf"), float("nan"), torch.finfo(dt).max, 1.0, -float("inf")]):
        A[0, i, i::7] = v                       # one value of K per row
        B[0, i, :] = torch.tensor([1.0, 2.0, -0.0, 3.0], dtype=dt).repeat(N // 4)
    fast = run_gpu(g, w, A, B, None, out_dtype="f32")
    slow = run_gpu(g, w, A, B, None, out_dtype="f32", config=g.config_names().index("general_mfma32_64x64x16"))
    assert torch.equal(torch.isnan(fast), torch.isnan(slow))
    assert torch.equal(torch.nan_to_num(fast, nan=0.5), torch.nan_to_num(slow, nan=0.5))


@pytest.mark.parametrize("la,lb", PAIRS)
@pytest.mark.parametrize("M,N,batch", [(72, 136, 3), (136, 200, 5), (264, 72, 8), (40, 264, 8)])
def test_batches_one_tile_per_workgroup(g, oracle, la, lb, M, N, batch):
    """Every one-tile-per-workgroup kernel over a batch with a bias: a tile count that is a multiple of 8 gives the deep
    kernels one grid over all problems (whole problems per XCD), any other one a grid row per problem."""
    for cfg in configs(g, False):
        w = wl.Workload("t", M, N, 200, layout_a=la, layout_b=lb, batch=batch, epilogue="bias_relu", seed_a=M, seed_b=N + 1)
        info = exact(g, oracle, w, cfg, out_dtype="f32", pad_a=8, pad_c=1)
        bm, bn = (int(x) for x in cfg.split("_")[1].split("x")[:2])
        tiles = -(-M // bm) * -(-N // bn)
        one_grid = cfg[-3:] in ("_s4", "_s5") and tiles * batch % 8 == 0
        assert (f"grid={tiles * batch},1,1" if one_grid else f"grid={tiles},{batch},1") in info, info


@pytest.mark.parametrize("la,lb", PAIRS)
def test_two_launches_and_their_unaligned_fallback(g, oracle, la, lb):
    """A plan whose last columns are a second launch (the offset into B depends on its layout): exact across the seam, and
    one kernel for all columns where A or B is only element-aligned."""
    w = wl.Workload("t", 1024, 17416, 136, layout_a=la, layout_b=lb, epilogue="bias_relu", seed_a=3, seed_b=4, seed_bias=5)
    info = exact(g, oracle, w, None, out_dtype="f32", pad_c=8)
    assert " + kernel=mfma16t_" in info and "columns=16384.." in info, info
    exact(g, oracle, w, None, offset_a=1)
    exact(g, oracle, w, None, offset_b=5)
