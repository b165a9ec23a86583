"""The skinny kernel with x in registers (skinnydirect_d2_b512_w4_rows) and the one beside it that fetches x from L2: exact on small
integers at the edges of the former's parts of K, of its panels of 16 rows and of the rule that chooses it, whichever of the two the rule
takes; values that are not finite stay in their own outputs; errors on normal data."""
import pytest
import torch

import workloads as wl
from test_gpu_wide_tiles import run_exact

pytestmark = pytest.mark.gpu
CFG, ROWS = "skinnydirect_d2_b512_w4", "skinnydirect_d2_b512_w4_rows"


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


# parts of K: one to four slabs, full, one piece short of full, one piece into the next; the last part short or empty
@pytest.mark.parametrize("K", [1032, 1536, 2040, 2048, 2056, 3592, 4096, 4104, 6136, 6144, 6152, 8184, 8192, 8200])
def test_parts_and_panels(g, K):
    for M, N in [(16, 16), (2, 17), (9, 1000), (5, 4113), (16, 8193)] + [(3, 12289)] * (K in (2056, 4096)) + [(16, 16401)] * (K < 2000):
        w = wl.Workload("t", M, N, K, epilogue="bias_relu", seed_a=K, seed_b=N)
        run_exact(g, w, CFG, out_dtype="f32")
        if N < 8000:
            run_exact(g, w, CFG, pad_c=3)


def test_fp16_and_the_rule(g):
    def block(**kw):
        p = g.gemm_create(g.GemmDesc(**kw))
        info = p.info()
        g.gemm_destroy(p)
        assert CFG in info
        return "block=512" in info
    assert block(M=16, N=28672, K=8192) and block(M=2, N=16, K=1032) and block(M=16, N=8192, K=4096)
    assert not block(M=16, N=8192, K=8192) and not block(M=16, N=4096, K=1024) and not block(M=16, N=28672, K=8200)
    assert not block(M=16, N=15, K=4096) and not block(M=16, N=4096, K=4096, batch=2)
    for M, N, K in [(7, 2000, 1400), (16, 9000, 2824)]:
        run_exact(g, wl.Workload("t", M, N, K, dtype="f16", epilogue="bias_relu", seed_a=K, seed_b=N), CFG)


@pytest.mark.parametrize("K", [1416, 4096, 5000])
def test_values_that_are_not_finite(g, K):
    M, N = 5, 3001 if K < 2048 else 9001
    A = torch.ones(M, K, dtype=torch.bfloat16, device="cuda")
    B = torch.ones(N, K, dtype=torch.bfloat16, device="cuda")
    want = torch.full((M, N), float(K))
    for row, col, v in [(0, 0, float("inf")), (1, K - 1, float("-inf")), (17, K // 2, float("nan")), (N - 1, K - 8, float("inf")), (N - 2, 0, float("nan"))]:
        B[row, col] = v
        want[:, row] = v
    A[M - 1, K - 1] = float("inf")
    want[M - 1] = torch.where(want[M - 1].isfinite(), float("inf"), want[M - 1])
    want[M - 1, 1] = float("-inf")
    C = torch.empty(M, N, device="cuda")
    p = g.gemm_create(g.GemmDesc(M, N, K, dtype_c=g.F32))
    assert "block=512" in p.info()
    g.gemm_run(p, A, B, C, None)
    torch.cuda.synchronize()
    g.gemm_destroy(p)
    want[M - 1, 1] = float("-inf")          # inf * -inf at the last column
    assert torch.equal(C.cpu().nan_to_num(nan=1e9, posinf=2e9, neginf=-2e9), want.nan_to_num(nan=1e9, posinf=2e9, neginf=-2e9))


@pytest.mark.parametrize("K", [1032, 1536, 2040, 2048, 2056, 3592, 4096, 4104, 6136, 6144, 6152, 8184, 8192])
def test_parts_and_panels_on_the_kernel_by_name(g, K):
    """The products of test_parts_and_panels on the kernel with x in registers, whichever of the two the rule takes."""
    for M, N in [(16, 16), (2, 17), (9, 1000), (5, 4113), (16, 8193)] + [(3, 12289)] * (K in (2056, 4096)) + [(16, 16401)] * (K < 2000):
        w = wl.Workload("t", M, N, K, epilogue="bias_relu", seed_a=K, seed_b=N)
        run_exact(g, w, ROWS, out_dtype="f32")
        if N < 8000:
            run_exact(g, w, ROWS, pad_c=3)


def test_fp16_and_the_rule_by_name(g):
    for kw, rows in ((dict(M=16, N=28672, K=8192), True), (dict(M=2, N=16, K=1032), True), (dict(M=16, N=8192, K=4096), True),
                     (dict(M=16, N=8192, K=8192), False), (dict(M=16, N=4096, K=1024), False), (dict(M=16, N=28672, K=8200), False)):
        p = g.gemm_create(g.GemmDesc(**kw))
        assert (ROWS in p.info()) == rows, p.info()
        g.gemm_destroy(p)
    for M, N, K in [(7, 2000, 1400), (16, 9000, 2824)]:
        run_exact(g, wl.Workload("t", M, N, K, dtype="f16", epilogue="bias_relu", seed_a=K, seed_b=N), ROWS)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K", [1032, 2048, 4104, 8192])
def test_error_on_normal_data(g, dtype, K):
    """32 products per addition into the accumulator and roundings inside: bound at 2^-24 sqrt(K / 32), as for the tiled kernels (eight parts
    of K add to it in fp32, each at most an eighth as long a sum)."""
    M, N = 16, 1000
    gen = torch.Generator(device="cuda:0").manual_seed(K)
    A, B = (torch.randn(r, K, generator=gen, device="cuda:0").to(wl.TORCH_DTYPE[dtype]) for r in (M, N))
    ref = A.double() @ B.double().t().contiguous()
    code = {"bf16": g.BF16, "f16": g.F16}[dtype]
    for cfg in (CFG, ROWS):
        C = torch.full((M, N), float("nan"), device="cuda:0")
        p = g.gemm_create_config(g.GemmDesc(M, N, K, dtype=code, dtype_c=g.F32), g.config_names().index(cfg))
        g.gemm_run(p, A, B, C)
        torch.cuda.synchronize()
        g.gemm_destroy(p)
        e = float((C.double() - ref).norm() / ref.norm())
        print(f"{dtype} K={K} {cfg}: {e:.2e}", flush=True)
        assert e <= 2.0 ** -24 * (K / 32) ** 0.5, (cfg, e)
