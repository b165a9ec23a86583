"""Which kernel a 16-bit product gets that is not K-contiguous in both operands: decided on the host, no GPU needed."""
import pytest

import paper_2603_12440_amd as g


def info(**kw):
    p = g.gemm_create(g.GemmDesc(**kw))
    text = p.info()
    g.gemm_destroy(p)
    return text


TILED = [dict(M=776, N=1032, K=456, layout_b=g.ROW_MAJOR), dict(M=776, N=1032, K=3001, layout_a=g.COL_MAJOR, layout_b=g.ROW_MAJOR),
         dict(M=776, N=1033, K=456, layout_a=g.COL_MAJOR), dict(M=777, N=1032, K=456, layout_b=g.ROW_MAJOR, dtype=g.F16),
         dict(M=776, N=1032, K=456, layout_b=g.ROW_MAJOR, batch=5, ldc=1033, dtype_c=g.F32)]
GENERAL = [dict(M=776, N=1033, K=456, layout_b=g.ROW_MAJOR), dict(M=776, N=1032, K=457, layout_b=g.ROW_MAJOR),
           dict(M=777, N=1032, K=456, layout_a=g.COL_MAJOR), dict(M=776, N=1032, K=456, layout_b=g.ROW_MAJOR, ldb=1033),
           dict(M=776, N=1032, K=456, layout_b=g.ROW_MAJOR, batch=2, stride_b=1032 * 456 + 4),
           dict(M=776, N=1032, K=456, layout_b=g.ROW_MAJOR, layout_c=g.COL_MAJOR),
           dict(M=776, N=1032, K=456, layout_b=g.ROW_MAJOR, dtype=g.F32)]


@pytest.mark.parametrize("kw", TILED)
def test_tiled(kw):
    """16-byte pieces along every operand's contiguous index; other pointers have a general kernel in the same plan."""
    text = info(**kw)
    assert "kernel=mfma16t_" in text and " unaligned A or B: kernel=" in text


@pytest.mark.parametrize("kw", GENERAL)
def test_general(kw):
    assert "mfma16t_" not in info(**kw)


def test_refusals_are_unchanged():
    """The K-contiguous configurations still refuse these layouts, the new ones refuse everything else."""
    names = g.config_names()
    for kw, prefixes in ((TILED[0], ("mfma_", "mfma16_", "skinny", "mfma8")), (dict(M=256, N=256, K=256), ("mfma16t_",)),
                         (GENERAL[0], ("mfma16t_",))):
        for i, n in enumerate(names):
            if n.startswith(prefixes):
                with pytest.raises(g.GemmError) as e:
                    g.gemm_create_config(g.GemmDesc(**kw), i)
                assert e.value.status == -9
    with pytest.raises(g.GemmError) as e:            # more rows than the general kernels' grid holds
        g.gemm_create(g.GemmDesc(1 << 30, 8, 8, layout_b=g.ROW_MAJOR))
    assert e.value.status == -2
    with pytest.raises(g.GemmError):
        g.gemm_create_splitk(g.GemmDesc(512, 512, 32768, layout_b=g.ROW_MAJOR), 0)


@pytest.mark.parametrize("dtype", [g.BF16, g.F16, g.F8E4M3])
def test_splitk_takes_whole_pieces_only(dtype):
    """Every slice's rows start on 16-byte pieces, whatever kernels serve other alignments in gemm_create."""
    def status(splits=0, **kw):
        try:
            p = g.gemm_create_splitk(g.GemmDesc(512, 512, 32768, dtype=dtype, **kw), splits)
        except g.GemmError as e:
            return e.status
        assert "+mfma16_" in p.info() or "+mfma8_" in p.info(), p.info()
        g.gemm_destroy(p)
        return 0
    for splits in (0, 1, 16):
        assert status(splits) == 0 and status(splits, lda=32768 + 16, ldb=32768 + 48) == 0
        assert status(splits, ldc=513) == 0 and status(splits, layout_c=g.COL_MAJOR) == 0      # (C is the reduction's)
        for kw in (dict(lda=32769), dict(ldb=32769), dict(lda=32768 + 4), dict(ldb=32768 + 4)):
            assert status(splits, **kw) == -4, (splits, kw)
        assert status(splits, lda=1 << 26) == -4                  # a tile's rows beyond 32-bit offsets


@pytest.mark.parametrize("M,N,K,dtype,slices", [
    (874, 2559, 17320, g.BF16, 1), (520, 3489, 14120, g.BF16, 1), (1057, 2840, 120504, g.F16, 1), (190, 3698, 122880, g.F16, 5),
    (2983, 3491, 77696, g.F16, 2), (3779, 2212, 14784, g.F16, 3), (314, 537, 512, g.F16, 2), (25, 3217, 512, g.F16, 4),
    (226, 686, 512, g.BF16, 2), (65, 1617, 512, g.F8E4M3, 4), (1160, 177, 512, g.F8E4M3, 2), (512, 512, 32768, g.BF16, 16)])
def test_number_of_slices(M, N, K, dtype, slices):
    """The library's own number of slices fixes the workspace, whether the fixed scratch buffer (32 MiB) holds it and the length
    of the fp32 sums: it stays what it is when tiles or the estimates behind gemm_create's choice change.  (Sizes at which
    tiles of 192 and 224 rows or a short-K term would move it, four of them across 32 MiB.)"""
    p = g.gemm_create_splitk(g.GemmDesc(M, N, K, dtype=dtype))
    assert f"kernel=splitk_{slices}+" in p.info() and g.gemm_workspace_bytes(p) == slices * M * N * 4
    g.gemm_destroy(p)


def fp32_lds(tile, M, N, K, **kw):
    p = g.gemm_create_config(g.GemmDesc(M, N, K, dtype=g.F32, layout_b=g.ROW_MAJOR, **kw), g.config_names().index(f"f32mfma_{tile}x{tile}x32"))
    lds = int(p.info().split(" lds=")[1].split()[0])
    g.gemm_destroy(p)
    return lds


# slabs of 32 columns of K: straight to LDS, 128 bytes a row, three of 64 + 64 rows or two of 128 + 128; or staged through
# registers, two slabs of rows of 36 values (K contiguous) and of 32 rows padded by 4
STRAIGHT = {64: 3 * 128 * 128, 128: 2 * 256 * 128}
STAGED = {tile: 2 * 4 * (tile * 36 + 32 * (tile + 4)) for tile in (64, 128)}


@pytest.mark.parametrize("tile", [64, 128])
def test_fp32_plans_report_the_lds_of_the_kernel_they_run(tile):
    assert fp32_lds(tile, 2000, 1500, 1100) == STRAIGHT[tile]
    assert fp32_lds(tile, 2000, 1500, 1100, lda=1 << 24) == STAGED[tile]       # offsets beyond 32 bits


def test_fp32_kernel_with_a_short_k():
    """64x64 tiles, 256 CUs: four workgroups of the staged kernel fit a CU, three of the other; tiles per CU beside each."""
    for M, N, K, batch, want in ((896, 4096, 32, 1, STAGED), (896, 4096, 36, 1, STAGED), (896, 4096, 192, 1, STAGED), (896, 4096, 196, 1, STRAIGHT),  # 3.5
                                 (768, 4096, 4, 1, STRAIGHT), (769, 4096, 4, 1, STAGED), (1024, 4096, 64, 1, STAGED), (1028, 4096, 4, 1, STRAIGHT),    # 3, 3.25, 4, 4.25
                                 (128, 192, 4, 128, STRAIGHT), (128, 192, 64, 150, STAGED), (64, 64, 4, 1, STRAIGHT),                                  # 3, 3.5, 0
                                 (1792, 4096, 32, 1, STAGED), (1792, 4096, 36, 1, STRAIGHT), (1536, 4096, 32, 1, STRAIGHT)):                           # 7, 7, 6
        assert fp32_lds(64, M, N, K, batch=batch) == want[64], (M, N, K, batch)
    assert fp32_lds(128, 896, 4096, 4) == STRAIGHT[128]


@pytest.mark.parametrize("kw,kernel", [
    (dict(M=613, N=21, K=15, batch=127), "general_mfma32_64x64x16"),               # 7.8 us; any-alignment tiles 15.0 and 19.2
    (dict(M=2319, N=879, K=9, layout_c=g.COL_MAJOR), "general_mfma32_64x64x16"),   # 7.2; 8.5 and 10.4
    (dict(M=697, N=41, K=37, batch=107), "mfma16g_64x64_k1_w2x2"),                 # 20.5; 24.9 with the larger tile
    (dict(M=4951, N=2497, K=65), "mfma16g_"), (dict(M=4951, N=2497, K=613), "mfma16g_128x128_k1_w2x4")])
def test_any_alignment_with_a_short_k(kw, kernel):
    """Up to 64 values of K the general kernel and the two any-alignment tiles are weighed against each other."""
    assert "kernel=" + kernel in info(**kw)
    if "batch" not in kw:
        assert "kernel=" + kernel in info(dtype_c=g.F32, **kw)


@pytest.mark.parametrize("kw,kernel", [
    (dict(M=387, N=104, K=32, batch=202), "mfma16_128x128x64_w2x2"),               # 10.4 us; 64x64 ring 19.2
    (dict(M=525, N=72, K=40, batch=233), "mfma16_128x128x64_w2x2"),                # 14.2; 24.2
    (dict(M=699, N=311, K=144, batch=46), "mfma16_128x128x64_w2x2"),               # 21.9; 64x64 ring 26.5
    (dict(M=413, N=340, K=48, batch=139), "mfma16_128x128x64_w2x2"),               # 23.7; 224x256 31.0
    (dict(M=1092, N=12052, K=312, dtype=g.F16, dtype_c=g.F32), "mfma16_224x256x64_w2x4"),    # 26.4; 128x128 36.9
    (dict(M=3422, N=8920, K=408, dtype_c=g.F32), "mfma16_2"),                      # tiles of 256 columns 59.4; 128x128 69.7
    (dict(M=3399, N=11442, K=6256), "mfma16_224x256x64_w2x4"),                     # 494; 128x128 625
    (dict(M=476, N=2077, K=10840), "mfma16_64x64_k1_w2x4_s5")])                    # 93; 128x128, four slabs 127
def test_choice_among_tiles(kw, kernel):
    """Products at which the estimate has to see a batch, a short K, fp32 results or a partial round as they are (us on one box)."""
    assert "kernel=" + kernel in info(**kw)


@pytest.mark.parametrize("M,N", [(6528, 6240), (1024, 17416), (2048, 12000)])
def test_choice_does_not_step_with_k(M, N):
    """K from 448 to 576: whole slabs on one tile, and others on one tile."""
    assert len({info(M=M, N=N, K=k).split()[0] for k in range(448, 577, 64)}) == 1
    assert len({info(M=M, N=N, K=k).split()[0] for k in range(448, 577, 8) if k % 64}) == 1


def test_second_launch_of_a_wide_product():
    """One launch, or whole rounds on 256x256 tiles and the rest as a second one: as measured."""
    for kw, two in ((dict(M=2048, N=14336, K=2048), False),                        # 92.2 us; 95.1 in two
                    (dict(M=4096, N=14336, K=4096, dtype=g.F8E4M3), True), (dict(M=4096, N=4608, K=4096), True),
                    (dict(M=1024, N=17416, K=136, layout_b=g.ROW_MAJOR, dtype_c=g.F32), True),     # 29.0; 31.7 in one
                    (dict(M=1024, N=17416, K=136, layout_b=g.ROW_MAJOR), False)):                  # 24.5; 25.5 in two
        assert ("columns=" in info(**kw)) == two, kw


@pytest.mark.parametrize("kw,kernel", [
    (dict(M=10, N=7, K=26, batch=294, layout_a=g.COL_MAJOR, layout_b=g.ROW_MAJOR), "general_mfma32_64x64x16"),       # 6.8 us; 16x16 tiles 8.4
    (dict(M=32, N=32, K=2000, batch=512), "f32mfma_64x64x32"),                     # 72.0; 16x16 tiles 105
    (dict(M=1079, N=467, K=529), "general_mfma32_64x64x16"),                       # 21.8; 33
    (dict(M=2456, N=110, K=2930, layout_b=g.ROW_MAJOR), "f32small_16x16x256"),     # 81; 117
    (dict(M=96, N=2, K=408, batch=139), "f32small_16x16x256"),                      # 9.9; 20.1
    (dict(M=4, N=208, K=2132, batch=70, layout_a=g.COL_MAJOR), "f32small_16x16x256"),                     # 45; 79
    (dict(M=4, N=584, K=300, batch=26, layout_a=g.COL_MAJOR, layout_b=g.ROW_MAJOR), "f32mfma_64x64x32"),
    (dict(M=139, N=1, K=7, batch=508), "f32general_64x64x16"),                     # 6.8; any-alignment kernel 9.3 and 14.0
    (dict(M=139, N=1, K=27, batch=508), "general_mfma32_64x64x16"), (dict(M=139, N=1, K=69, batch=508), "f32general_64x64x16")])
def test_fp32_choice(kw, kernel):
    """fp32 products between one and two 32x32 tiles per CU, and narrow ones of any alignment in large numbers (us on one box)."""
    assert "kernel=" + kernel + " " in info(dtype=g.F32, **kw)


def by_name(name, **kw):
    p = g.gemm_create_config(g.GemmDesc(**kw), g.config_names().index(name))
    text = p.info()
    g.gemm_destroy(p)
    return text


@pytest.mark.parametrize("tile,shape", [("256x256", "w2x4"), ("224x256", "w2x4"), ("192x256", "w2x4"), ("256x192", "w4x2"), ("128x128", "w2x2")])
def test_fp8_tiles_with_and_without_persistent_workgroups(tile, shape):
    """Both kernels of an fp8 tile have a name, whatever K is (_s2: persistent workgroups where K is two or more whole slabs of 128)."""
    bm, bn = (int(x) for x in tile.split("x"))
    name = f"mfma8_{tile}x128_{shape}_"
    kw = dict(M=20 * bm, N=40 * bn, dtype=g.F8E4M3)
    assert f"grid={512 if tile == '128x128' else 256},1,1" in by_name(name + "s2", K=512, **kw)
    for k in (512, 528, 128):
        assert "grid=800,1,1" in by_name(name + "one", K=k, **kw)
    assert "grid=800,1,1" in by_name(name + "s2", K=528, **kw) and "grid=800,1,1" in by_name(name + "s2", K=128, **kw)


def test_fp8_choice_names_the_kernel_that_runs():
    """A K that is no whole number of slabs: one tile per workgroup."""
    for k in (144, 272, 1040, 4112):
        text = info(M=4096, N=8192, K=k, dtype=g.F8E4M3)
        assert "_s2 " not in text and ("_one " in text or "_s4 " in text or "_s5 " in text), text
    assert "_s2 " in info(M=8192, N=8192, K=8192, dtype=g.F8E4M3)


def test_both_skinny_kernels_have_a_name():
    """x in registers (panels of 16 rows of W, one workgroup of eight waves per CU) and x from L2 (panels of 32, four waves): either can be
    asked for where the built-in choice takes the other."""
    direct, rows = "skinnydirect_d2_b512_w4", "skinnydirect_d2_b512_w4_rows"
    for kw in (dict(M=16, N=8192, K=8192), dict(M=4, N=28672, K=4096), dict(M=9, N=1000, K=1032)):
        assert "tile=16x32x256" in by_name(direct, **kw) and "block=256 lds=65536" in by_name(direct, **kw)
        assert "tile=16x16x256" in by_name(rows, **kw) and "block=512 lds=81920" in by_name(rows, **kw)
    assert f"kernel={direct} " in info(M=16, N=8192, K=8192) and f"kernel={rows} " in info(M=16, N=28672, K=8192)
    for kw in (dict(M=16, N=8192, K=1024), dict(M=16, N=8192, K=8200), dict(M=16, N=15, K=4096), dict(M=16, N=4096, K=4096, batch=2),
               dict(M=17, N=4096, K=4096), dict(M=16, N=4096, K=4096, dtype=g.F8E4M3)):
        with pytest.raises(g.GemmError) as e:
            by_name(rows, **kw)
        assert e.value.status == -9, kw


def field(text, name):
    return text.split(" " + name + "=")[1].split()[0]


@pytest.mark.parametrize("tile", [64, 128])
def test_plans_of_any_alignment_report_the_kernel_they_run(tile):
    """fp32: slabs of 32 columns of K and two stages of 128 bytes a row, or, where offsets inside a slab do not fit 32 bits and on
    f32general_64x64x16, the general kernel's 16 columns."""
    name, general = f"general_mfma32_{tile}x{tile}x16", 4 * 16 * 2 * (tile + 4)
    kw = dict(M=1001, N=1001, K=1001, dtype=g.F32)
    last = ((1 << 32) - 1) // (4 * (tile + 1)) // 4 * 4                           # (tile + 1) rows below 2^32 bytes
    for extra, k, lds in ((dict(), 32, 512 * tile), (dict(lda=last), 32, 512 * tile), (dict(lda=last + 4), 16, general), (dict(ldb=last + 4), 16, general)):
        text = by_name(name, **kw, **extra)
        assert field(text, "tile") == f"{tile}x{tile}x{k}" and int(field(text, "lds")) == lds, (extra, text)
    assert field(by_name(name, M=1001, N=1001, K=1001), "tile") == f"{tile}x{tile}x16"       # 16-bit operands
    if tile == 64:
        assert field(by_name("f32general_64x64x16", **kw), "tile") == "64x64x16" and int(field(by_name("f32general_64x64x16", **kw), "lds")) == general


def test_two_launches_and_slices_report_the_lds_of_the_kernel_they_run():
    """Slabs of 256 + 256 rows of 128 bytes, two of them; a persistent workgroup's staging area or 256 bytes behind them."""
    slabs = 2 * 512 * 128
    for k, lds in ((4096, slabs + 32768), (4112, slabs + 256)):
        text = info(M=4096, N=14336, K=k, dtype=g.F8E4M3)
        assert "mfma8_256x256x128" in text and int(field(text, "lds")) == lds, text
    assert int(field(by_name("mfma8_256x256x128_w2x4_s2", M=4096, N=14336, K=4112, dtype=g.F8E4M3), "lds")) == slabs + 256
    for M, N, K, slices, dtype in ((512, 512, 32768, 16, g.BF16), (512, 512, 32768, 16, g.F8E4M3), (2048, 2048, 16 * 1040, 4, g.F8E4M3)):
        p = g.gemm_create_splitk(g.GemmDesc(M, N, K, dtype=dtype), slices)
        name = p.info().split("+")[1].split()[0]
        inner = by_name(name, M=M, N=N, K=K // slices, dtype=dtype, dtype_c=g.F32)
        assert field(p.info(), "lds") == field(inner, "lds") and field(p.info(), "tile") == field(inner, "tile"), (p.info(), inner)
        g.gemm_destroy(p)
