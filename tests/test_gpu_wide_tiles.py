"""The eight-wave tiles 192x256, 224x256 and 256x256 (16-bit operands): exact on small integers in every layout, around the
hand-over of the first and last slabs, K tails, ragged tiles, and persistent workgroups that walk over several tiles."""
import pytest
import torch

import workloads as wl
from helpers import gpu_desc, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


def run_exact(g, w, cfg, **kw):
    """Against fp32 torch on the host: sums of small integers are exact in any order."""
    A = wl.small_integers(wl.operand_shapes(w)[0], w.seed_a, -1, 1, w.dtype)
    B = wl.small_integers(wl.operand_shapes(w)[1], w.seed_b, -1, 1, w.dtype)
    bias = wl.small_integers((w.N,), w.seed_bias, -3, 3, "f32") if w.has_bias else None
    print(f"{w.M}x{w.N}x{w.K} b{w.batch} {w.dtype} {w.layout_a}/{w.layout_b} {cfg}", flush=True)
    C = run_gpu(g, w, A, B, bias, config=g.config_names().index(cfg), **kw)
    a = A.float() if w.layout_a == "row" else A.float().transpose(1, 2).contiguous()
    b = B.float() if w.layout_b == "row" else B.float().transpose(1, 2).contiguous()
    want = torch.matmul(a, b)
    if bias is not None:
        want = torch.relu(want + bias)
    assert torch.equal(C.float(), want.to(C.dtype).float()), cfg


def configs(g, la, lb):
    family = "mfma16_" if (la, lb) == ("row", "col") else "mfma16t_"
    return [n for n in g.config_names() if n.startswith(tuple(family + f"{bm}x256x64_w2x4" for bm in (192, 224, 256)))]


@pytest.mark.parametrize("la,lb", [("row", "col"), ("row", "row"), ("col", "row"), ("col", "col")])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_slabs_tails_and_edges(g, dtype, la, lb):
    """One slab to several, with and without a tail of one or two k-steps; rows just below, at and above a tile.
    (|sum| <= 648 + 3: exact in fp32 output; bf16 output is the same rounding of the same value.)"""
    names = configs(g, la, lb)
    assert len(names) >= 4
    for cfg in names:
        bm = int(cfg.split("_")[1].split("x")[0])
        for M, N, K in ((bm, 256, 64), (bm - 8, 264, 128), (bm + 8, 248, 192), (8, 8, 256), (bm, 512, 320), (2 * bm + 16, 264, 640),
                        (bm + 32, 40, 8), (bm - 24, 256, 72), (2 * bm, 264, 104), (bm + 8, 256, 168), (3 * bm - 8, 520, 200), (200, 264, 648)):
            if cfg.endswith("_p") and (K % 64 or K < 128):
                continue
            w = wl.Workload("t", M, N, K, dtype=dtype, layout_a=la, layout_b=lb, epilogue="bias_relu", seed_a=K, seed_b=M)
            run_exact(g, w, cfg, out_dtype="f32")
            run_exact(g, w, cfg)
        for N in (257, 519):                                # rows of C that start at any element
            w = wl.Workload("t", bm + 8, N if lb == "col" else N // 8 * 8, 256, dtype=dtype, layout_a=la, layout_b=lb, epilogue="bias_relu", seed_a=N, seed_b=3)
            run_exact(g, w, cfg, pad_c=1)
            run_exact(g, w, cfg, pad_c=3, out_dtype="f32")
        run_exact(g, wl.Workload("t", bm + 8, 264, 192, dtype=dtype, layout_a=la, layout_b=lb, batch=3, seed_a=1, seed_b=2), cfg, out_dtype="f32")


@pytest.mark.parametrize("la,lb", [("row", "col"), ("row", "row"), ("col", "row"), ("col", "col")])
def test_several_tiles_per_workgroup(g, la, lb):
    """More tiles than CUs, in numbers that divide by 8 and that do not, and a batch."""
    for cfg in (n for n in configs(g, la, lb) if n.endswith("_p")):
        for M, N, K, batch in ((3000, 6000, 128, 1), (2304, 8192, 192, 1), (504, 1000, 256, 41)):
            run_exact(g, wl.Workload("t", M, N, K, dtype="bf16", layout_a=la, layout_b=lb, batch=batch, seed_a=K, seed_b=N), cfg)


@pytest.mark.parametrize("la,lb", [("row", "col"), ("row", "row"), ("col", "row"), ("col", "col")])
def test_few_tiles_along_a_panel(g, la, lb):
    """One to five tile rows or columns, where workgroups share the lines they prefetch among fewer than four or eight."""
    for cfg in configs(g, la, lb):
        bm = int(cfg.split("_")[1].split("x")[0])
        for tiles_m, tiles_n, K in ((1, 1, 256), (1, 5, 320), (2, 3, 256), (3, 1, 192), (5, 2, 448)):
            run_exact(g, wl.Workload("t", tiles_m * bm - 8, tiles_n * 256 - 16, K, dtype="bf16", layout_a=la, layout_b=lb, seed_a=K, seed_b=tiles_n), cfg)


def test_built_in_choice(g):
    """A wide tile where it fills the CUs better than 256x256."""
    for M, N, K, la, lb, want in ((3001, 4096, 6144, "row", "row", "192x256"), (777, 14336, 4096, "row", "col", "224x256"),
                                  (6144, 4096, 3001, "col", "row", "192x256"), (8192, 8192, 8192, "row", "col", "256x256")):
        info = g.gemm_plan_info(g.gemm_create(gpu_desc(g, wl.Workload("t", M, N, K, dtype="bf16", layout_a=la, layout_b=lb), None)))
        assert want in info, info
