"""fp32 products of any extent and alignment (16-byte loads at four-byte alignment): bit exact on small integers for every layout around
tile edges, slabs and the last piece of K; pointers at any element; values that are not finite stay in their own outputs."""
import pytest
import torch

import workloads as wl
from helpers import gpu_desc, run_gpu

pytestmark = pytest.mark.gpu
LAYOUTS = [("row", "row"), ("row", "col"), ("col", "row"), ("col", "col")]
CFGS = ("general_mfma32_64x64x16", "general_mfma32_128x128x16", "f32small_16x16x256")


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


def operands(w):
    A = wl.small_integers(wl.operand_shapes(w)[0], w.seed_a, -2, 2, "f32")
    B = wl.small_integers(wl.operand_shapes(w)[1], w.seed_b, -2, 2, "f32")
    a = A if w.layout_a == "row" else A.transpose(1, 2).contiguous()
    b = B if w.layout_b == "row" else B.transpose(1, 2).contiguous()
    return A, B, torch.matmul(a, b)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("M,N,K,batch", [(1, 1, 1, 1), (3, 2, 3, 1), (5, 66, 4, 1), (63, 65, 31, 1), (64, 64, 33, 1), (65, 127, 34, 1), (129, 131, 63, 1),
                                         (127, 193, 65, 2), (130, 130, 67, 3), (257, 61, 130, 1), (17, 333, 257, 1), (20, 35, 515, 1), (40, 47, 1030, 5), (66, 62, 97, 8)])
def test_exact(g, la, lb, M, N, K, batch):
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, batch=batch, epilogue="bias_relu", seed_a=M + 1, seed_b=N + 2)
    A, B, want = operands(w)
    bias = wl.small_integers((N,), w.seed_bias, -3, 3, "f32")
    want = torch.relu(want + bias)
    for cfg in CFGS:
        for lc, pads in (("row", (0, 0, 0)), ("col", (1, 3, 1)), ("row", (2, 5, 2))):
            print(f"{M}x{N}x{K} b{batch} {la}/{lb}/{lc} {cfg} {pads}", flush=True)
            C = run_gpu(g, w, A, B, bias, config=g.config_names().index(cfg), layout_c=lc, pad_a=pads[0], pad_b=pads[1], pad_c=pads[2])
            assert torch.equal(C.float(), want), (cfg, lc, pads)


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_pointers_at_any_element(g, la, lb):
    M, N, K = 132, 200, 100
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, seed_a=1, seed_b=2)
    A, B, want = operands(w)
    for cfg in ("f32mfma_64x64x32", "f32mfma_128x128x32") + CFGS:
        p = g.gemm_create_config(gpu_desc(g, w), g.config_names().index(cfg))
        for oa, ob in ((1, 0), (0, 3), (2, 1)):
            print(la, lb, cfg, oa, ob, flush=True)
            a, b = torch.empty(A.numel() + oa, device="cuda"), torch.empty(B.numel() + ob, device="cuda")
            a[oa:], b[ob:] = A.flatten().cuda(), B.flatten().cuda()
            C = torch.full((M, N), -7.0, device="cuda")
            g.gemm_run(p, a[oa:], b[ob:], C, None)
            torch.cuda.synchronize()
            assert torch.equal(C.cpu(), want[0]), cfg
        g.gemm_destroy(p)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("K", [66, 261])
def test_values_that_are_not_finite(g, la, lb, K):
    M, N = 70, 133
    a, b = torch.ones(M, K), torch.ones(K, N)
    want = torch.full((M, N), float(K))
    for row, col, v in [(0, 0, float("inf")), (17, K - 1, float("nan")), (N - 1, K // 2, float("-inf")), (64, K - 2, float("inf"))]:
        b[col, row] = v
        want[:, row] = v
    a[M - 1, K - 1] = float("inf")
    want[M - 1] = torch.where(want[M - 1].isfinite(), float("inf"), want[M - 1])
    want[M - 1, N - 1] = float("nan")
    A = (a if la == "row" else a.t().contiguous()).cuda()
    B = (b if lb == "row" else b.t().contiguous()).cuda()
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb)
    for cfg in CFGS:
        C = torch.empty(M, N, device="cuda")
        p = g.gemm_create_config(gpu_desc(g, w), g.config_names().index(cfg))
        g.gemm_run(p, A, B, C, None)
        torch.cuda.synchronize()
        g.gemm_destroy(p)
        assert torch.equal(C.cpu().nan_to_num(nan=1e9, posinf=2e9, neginf=-2e9), want.nan_to_num(nan=1e9, posinf=2e9, neginf=-2e9)), cfg


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("M,N,K,batch", [(1100, 1030, 67, 1), (2100, 2200, 35, 1), (70, 130, 40, 70), (200, 24, 33, 150), (139, 1, 7, 508), (100, 49, 33, 300),
                                         (100, 30, 17, 200), (30, 49, 130, 300)])
def test_lanes_along_rows_and_columns(g, la, lb, M, N, K, batch):
    """More and fewer tiles than CUs, few columns and more, C in either layout: a lane holds values of a row or of a column of C."""
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, batch=batch, epilogue="bias_relu", seed_a=M + 1, seed_b=N + 2)
    A, B, want = operands(w)
    bias = wl.small_integers((N,), w.seed_bias, -3, 3, "f32")
    want = torch.relu(want + bias)
    for cfg in ("general_mfma32_64x64x16", "general_mfma32_128x128x16", "f32general_64x64x16", None):
        for lc in ("row", "col"):
            print(f"{M}x{N}x{K} b{batch} {la}/{lb}/{lc} {cfg}", flush=True)
            C = run_gpu(g, w, A, B, bias, config=-1 if cfg is None else g.config_names().index(cfg), layout_c=lc, pad_a=1, pad_c=1)
            assert torch.equal(C.float(), want), (cfg, lc)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("huge", ["a", "b"])
def test_offsets_at_and_beyond_32_bits(g, la, lb, huge):
    """A leading dimension at which 65 or 129 rows just fit 2^32 bytes, the next one in whole pieces, and 2^24: the kernel of 16-byte loads at any
    alignment, then the general one, on the plans of either tile and, with a pointer displaced by one element, on those for aligned pieces.
    (Two to five GB of address space, few rows touched.)"""
    M, N, K = 72, 68, 36
    w = wl.Workload("t", M, N, K, dtype="f32", layout_a=la, layout_b=lb, epilogue="bias_relu", seed_a=1, seed_b=2)
    A, B, want = operands(w)
    bias = wl.small_integers((N,), w.seed_bias, -3, 3, "f32")
    want = torch.relu(want + bias)
    Ad, Bd, biasd = A.cuda(), B.cuda(), bias.cuda()
    src = Ad if huge == "a" else Bd
    for ld in (8323580, 8323584, 16519104, 16519108, 1 << 24):
        wide = torch.empty((src.shape[1] - 1) * ld + src.shape[2] + 1, device="cuda")
        for off in (0, 1):
            rows = wide[off:].as_strided((src.shape[1], src.shape[2]), (ld, 1))
            rows.copy_(src[0])
            for cfg in ("general_mfma32_64x64x16", "general_mfma32_128x128x16", "f32general_64x64x16") + ("f32mfma_64x64x32", "f32mfma_128x128x32") * off:
                C = torch.full((M, N), -7.0, device="cuda")
                p = g.gemm_create_config(gpu_desc(g, w, **{"ld" + huge: ld}), g.config_names().index(cfg))
                print(f"{la}/{lb} {huge} ld={ld} + {off} {p.info()}", flush=True)
                g.gemm_run(p, rows if huge == "a" else Ad, rows if huge == "b" else Bd, C, biasd)
                torch.cuda.synchronize()
                g.gemm_destroy(p)
                assert torch.equal(C.cpu(), want[0]), (cfg, ld, off)


@pytest.mark.parametrize("M", [1, 8, 9])
@pytest.mark.parametrize("K", [1021, 1025, 1031])
def test_few_rows_and_a_long_k(g, M, K):
    """16x16 tiles, both operands row-major: A value by value up to eight rows with K > 1024, in groups beyond; at any element."""
    w = wl.Workload("t", M, 35, K, dtype="f32", layout_a="row", layout_b="row", batch=3, epilogue="bias_relu", seed_a=M, seed_b=K)
    A, B, want = operands(w)
    bias = wl.small_integers((35,), w.seed_bias, -3, 3, "f32")
    for pad in (0, 2):
        C = run_gpu(g, w, A, B, bias, config=g.config_names().index("f32small_16x16x256"), pad_a=pad, pad_b=pad)
        assert torch.equal(C.float(), torch.relu(want + bias)), pad
