"""The kernels whose waves split K, tiles of 64x64 and 32x32: exact on small integers around whole turns of the
waves, K tails, ragged tiles, batches and the rule that chooses it; values that are not finite stay in their own outputs."""
import pytest
import torch

import workloads as wl
from test_gpu_wide_tiles import run_exact

pytestmark = pytest.mark.gpu
C64, C32, K64x32 = "ksplit16_64x64_w8_s1", "ksplit16_32x32_w4_s4", "mfma16_64x32_k4_w4x2_s3"


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


def test_built_in_choice(g):
    def kernel(M, N, K, **kw):
        p = g.gemm_create(g.GemmDesc(M, N, K, **kw))
        info = p.info()
        g.gemm_destroy(p)
        return info
    assert C32 in kernel(96, 512, 2048) and C32 in kernel(17, 512, 4096) and C64 in kernel(512, 2048, 8192)
    for kw in (dict(M=96, N=512, K=1152), dict(M=17, N=512, K=2048), dict(M=96, N=512, K=2056), dict(M=4096, N=4096, K=2048)):
        assert "ksplit16" not in kernel(**kw), kw


# no slab, fewer slabs than waves, 22 to 25, then whole turns and a long K; tails in rows on 128-byte lines (pad)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K,pad", [(8, 56), (64, 0), (200, 56), (576, 0), (1408, 0), (1472, 64), (1536, 0), (1600, 0), (1416, 56), (1528, 8), (1592, 8), (1544, 56), (2048, 0), (4096, 0)])
def test_slabs_tails_and_edges(g, dtype, K, pad):
    for cfg, shapes in ((C64, [(200, 250), (256, 1024), (1001, 250)]), (C32, [(65, 100), (96, 96), (513, 320)]), (K64x32, [(33, 47), (128, 96)])):
        for M, N in shapes:
            w = wl.Workload("t", M, N, K, dtype=dtype, epilogue="bias_relu", seed_a=K, seed_b=M)
            run_exact(g, w, cfg, out_dtype="f32", pad_a=pad, pad_b=pad)
            run_exact(g, w, cfg, pad_a=pad, pad_b=pad, pad_c=3)
    w = wl.Workload("t", 70, 96, K, dtype=dtype, batch=8, seed_a=K, seed_b=4)
    run_exact(g, w, C32, out_dtype="f32", pad_a=pad, pad_b=pad)
    run_exact(g, wl.Workload("t", 193, 200, K, dtype=dtype, batch=3, seed_a=K, seed_b=4), C64, out_dtype="f32", pad_a=pad, pad_b=pad)


@pytest.mark.parametrize("cfg", [C64, C32])
@pytest.mark.parametrize("K,ld", [(1536, 1536), (1544, 1600)])
def test_values_that_are_not_finite(g, cfg, K, ld):
    M, N = 250, 300 if cfg == C64 else 130
    A = torch.full((M, ld), float("nan"), dtype=torch.bfloat16, device="cuda")     # (what lies behind K is never multiplied)
    B = torch.full((N, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    A[:, :K] = 1
    B[:, :K] = 1
    want = torch.full((M, N), float(K))
    for row, col, v in [(0, 0, float("inf")), (17, K - 1, float("nan")), (N - 1, 700, float("-inf"))]:
        B[row, col] = v
        want[:, row] = v
    A[M - 1, K - 1] = float("inf")
    want[M - 1] = torch.where(want[M - 1].isfinite(), float("inf"), want[M - 1])
    want[M - 1, N - 1] = float("nan")
    C = torch.empty(M, N, device="cuda")
    p = g.gemm_create_config(g.GemmDesc(M, N, K, lda=ld, ldb=ld, dtype_c=g.F32), g.config_names().index(cfg))
    g.gemm_run(p, A, B, C, None)
    torch.cuda.synchronize()
    g.gemm_destroy(p)
    assert torch.equal(C.cpu().nan_to_num(nan=1e9, posinf=2e9, neginf=-2e9), want.nan_to_num(nan=1e9, posinf=2e9, neginf=-2e9))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K", [1024, 4096])
def test_error_on_normal_data(g, dtype, K):
    """The same products as the tiled kernels, in as many sums as there are waves, added in fp32: within the tiled kernels' bound,
    2^-24 sqrt(K / 32) for 32 products per addition into the accumulator."""
    M, N = 136, 264
    gen = torch.Generator(device="cuda:0").manual_seed(K)
    A, B = (torch.randn(r, K, generator=gen, device="cuda:0").to(wl.TORCH_DTYPE[dtype]) for r in (M, N))
    ref = A.double() @ B.double().t().contiguous()
    code = {"bf16": g.BF16, "f16": g.F16}[dtype]
    for cfg in (C64, C32):
        C = torch.full((M, N), float("nan"), device="cuda:0")
        p = g.gemm_create_config(g.GemmDesc(M, N, K, dtype=code, dtype_c=g.F32), g.config_names().index(cfg))
        g.gemm_run(p, A, B, C)
        torch.cuda.synchronize()
        g.gemm_destroy(p)
        e = float((C.double() - ref).norm() / ref.norm())
        print(f"{dtype} K={K} {cfg}: {e:.2e}", flush=True)
        assert e <= 2.0 ** -24 * (K / 32) ** 0.5, (cfg, e)
