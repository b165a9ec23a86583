"""How far fp32 results are from 64 bits, kernel by kernel, on normal data.

Every product of two 16-bit or fp32 operands enters a sum kept in fp32.  For n dependent additions of random terms whose partial
sums grow like sqrt(i), each rounded to half a unit at random, the 2-norm of the error over that of the result is about
0.3 * 2^-24 * sqrt(n).  fp32 instruction: n = K, bound at 0.5.  16-bit matrix instruction: 32 products per addition into the
accumulator and roundings inside, measured at 0.52 to 0.58 * 2^-24 * sqrt(K / 32), bound at 1.  fp8 instruction: the products of
one step are added with fewer bits, 1.3e-5 whatever K is, bound at twice that.  So an error that doubled is noticed."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

M, N = 136, 264


@pytest.fixture(scope="module")
def g():
    import paper_2603_12440_amd as g
    g.load_library()
    assert torch.cuda.is_available()
    return g


def operands(dtype, K):
    gen = torch.Generator(device="cuda:0").manual_seed(K)
    A, B = (torch.randn(r, K, generator=gen, device="cuda:0").to(wl.TORCH_DTYPE[dtype]) for r in (M, N))
    return A, B, A.double() @ B.double().t().contiguous()


def run_all(g, dtype, K, A, B, layouts, wanted):
    """(layouts, configuration) -> fp32 C of every configuration that takes these layouts."""
    code = {"bf16": g.BF16, "f16": g.F16, "f8": g.F8E4M3, "f32": g.F32}[dtype]
    out = {}
    for la, lb in layouts:
        Al, Bl = A if la == g.ROW_MAJOR else A.t().contiguous(), B if lb == g.COL_MAJOR else B.t().contiguous()
        for i, name in enumerate(g.config_names()):
            if not name.startswith(wanted):
                continue
            pad = 1 if name.startswith("mfma16g_") else 0           # (that kernel takes what is not whole 16-byte pieces)
            Ap, Bp = (torch.nn.functional.pad(X, (0, pad)) if pad else X for X in (Al, Bl))
            try:
                plan = g.gemm_create_config(g.GemmDesc(M, N, K, dtype=code, layout_a=la, layout_b=lb, dtype_c=g.F32,
                                                       lda=Ap.shape[1], ldb=Bp.shape[1]), i)
            except g.GemmError:
                continue
            C = torch.full((M, N), float("nan"), device="cuda:0")
            print(f"{dtype} K={K} {la}{lb} {name}", flush=True)
            g.gemm_run(plan, Ap, Bp, C)
            torch.cuda.synchronize()
            g.gemm_destroy(plan)
            out[(la, lb, name)] = C
    return out


def error(C, ref):
    return float((C.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K", [328, 1024, 4096])
def test_16_bit_operands(g, dtype, K):
    """Every tiled kernel adds the same products in the same order, whatever its layout, tile and number of slabs: one result,
    bit for bit, no further off than the general kernel's fp32 products and sums."""
    A, B, ref = operands(dtype, K)
    both = [(a, b) for a in (g.ROW_MAJOR, g.COL_MAJOR) for b in (g.ROW_MAJOR, g.COL_MAJOR)]
    got = run_all(g, dtype, K, A, B, both, ("mfma16_", "mfma16t_", "mfma16g_", "mfma_"))
    assert len(got) >= 35, len(got)
    one = got[(g.ROW_MAJOR, g.COL_MAJOR, "mfma16_128x128x64_w2x2")]
    for key, C in got.items():
        assert torch.equal(C, one), key
    general = run_all(g, dtype, K, A, B, both[:1], ("general_mfma32_64x64x16",))
    assert error(one, ref) <= min(2.0 ** -24 * (K / 32) ** 0.5, *(error(C, ref) for C in general.values()))


@pytest.mark.parametrize("K", [320, 1024, 4096])
def test_8_bit_operands(g, K):
    A, B, ref = operands("f8", K)
    got = run_all(g, "f8", K, A, B, [(g.ROW_MAJOR, g.COL_MAJOR)], ("mfma8_",))
    assert len(got) >= 8, len(got)
    one = got[(g.ROW_MAJOR, g.COL_MAJOR, "mfma8_128x128x128_w2x2_s2")]
    for key, C in got.items():
        assert abs(error(C, ref) / error(one, ref) - 1) < 0.02, key
    assert error(one, ref) <= 2.7e-5


@pytest.mark.parametrize("K", [28, 328, 1024, 4096])
def test_32_bit_operands(g, K):
    A, B, ref = operands("f32", K)
    both = [(a, b) for a in (g.ROW_MAJOR, g.COL_MAJOR) for b in (g.ROW_MAJOR, g.COL_MAJOR)]
    got = run_all(g, "f32", K, A, B, both, ("f32mfma_", "f32small_", "general_mfma32_"))
    assert len(got) == 20, len(got)
    for key, C in got.items():
        assert error(C, ref) <= 0.5 * 2.0 ** -24 * K ** 0.5, (key, error(C, ref))
