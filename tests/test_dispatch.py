"""The kernel each rule of the dispatch picks, on both sides of its lines, by
the describe calls (host-side planning for 256 compute units, no GPU)."""
import re

import pytest

from paper_1810_11066_amd import bitserial as bs

U, B, S = bs.UNIPOLAR, bs.BIPOLAR, bs.SIGNED


@pytest.fixture(autouse=True)
def defaults():
    bs.load_library()
    yield
    bs.bs_set_kernel_mode(0)
    bs.bs_set_units_per_wave(0)


def conv(n, h, w, c, oc, k, s, abits, wbits, aenc=U, wenc=U):
    return bs.ConvParams(n, h, w, c, oc, k, k, s, s, k // 2, k // 2, abits,
                         wbits, aenc, wenc)


def dense(m, k, n, abits, wbits, aenc=U, wenc=U):
    return conv(1, 1, m, k, n, 1, 1, abits, wbits, aenc, wenc)


def family(p):
    return bs.bs_conv2d_describe(p).split("_kernel")[0]


def test_lone_waves():
    """At most one wave per SIMD, a workgroup per CU: the kernel for lone
    waves; one workgroup more: the kernel for several."""
    bs.bs_set_units_per_wave(1)
    for oc, lone in ((64, True), (68, False)):      # 1024 and 1088 units
        d = bs.bs_conv2d_describe(conv(16, 16, 16, 64, oc, 3, 1, 2, 2))
        assert d.startswith("conv_pix_kernel"), d
        assert d.endswith(" lone waves") == lone, d
    for oc, lone in ((64, True), (68, False)):
        d = bs.bs_conv2d_codes_describe(conv(16, 16, 16, 64, oc, 3, 1, 2, 2))
        assert d.endswith(" lone waves") == lone, d


@pytest.mark.parametrize("c,oc,k,abits,wbits,lone", [
    (32, 64, 3, 1, 1, True),       # 9 word pairs a result: stores bound it
    (32, 64, 3, 2, 1, False),      # 18
    (32, 732, 3, 2, 1, True),      # 18, rows end within a 64-byte piece
    (64, 732, 3, 2, 1, False),     # 36
    (128, 256, 1, 2, 1, True),     # 8
    (64, 256, 1, 4, 1, False),     # 8, 4-bit activations
    (32, 768, 1, 3, 3, False),     # 9, several filter planes
    (32, 724, 3, 1, 2, False),     # 18, of one activation plane
    (64, 732, 1, 3, 3, True),      # 18, of three
    (32, 732, 1, 3, 3, False),     # 9, of three and one word
])
def test_store_bound_results(c, oc, k, abits, wbits, lone):
    bs.bs_set_units_per_wave(1)
    d = bs.bs_conv2d_describe(conv(64, 28, 28, c, oc, k, 1, abits, wbits))
    assert d.startswith("conv_pix_kernel"), d
    assert d.endswith(" lone waves") == lone, d


@pytest.mark.parametrize("c,oc,k,lone", [
    (32, 64, 3, True), (32, 732, 3, True), (128, 256, 1, False),
    (128, 732, 1, True)])
def test_store_bound_staged(c, oc, k, lone):
    bs.bs_set_units_per_wave(1)
    p = conv(64, 28, 28, c, oc, k, 1, 2 if k == 1 else 1, 1)
    for describe in ([bs.bs_conv2d_codes_describe] +
                     [bs.bs_conv2d_quantized_describe] * (k == 1)):
        d = describe(p)
        assert d.endswith(" lone waves") == lone, d


@pytest.mark.parametrize("n,h,c,oc,k,abits,wbits,plan", [
    # 9 steps: waves share a unit's until there are 3 for every SIMD
    (48, 27, 96, 150, 3, 2, 1, "C=16> units=5470 of 16 waves=1"),
    (29, 27, 96, 150, 3, 2, 1, "C=16> units=3310 of 16 waves=1"),
    (26, 27, 96, 150, 3, 2, 1, "C=16> units=2970 of 16 waves=2"),
    # 18 steps: two until there are 4, four until there are 3.5
    (49, 20, 192, 192, 3, 2, 1, "C=16> units=3684 of 16 waves=2"),
    (55, 20, 192, 192, 3, 2, 1, "C=16> units=4128 of 16 waves=1"),
    (23, 20, 192, 192, 3, 2, 1, "C=16> units=1728 of 16 waves=4"),
    (25, 20, 192, 192, 3, 2, 1, "C=16> units=1884 of 16 waves=2"),
    # narrower units until there are 4
    (44, 20, 192, 192, 3, 3, 3, "C=4> units=6600 of 8 waves=1"),
    # 4-channel tiles below 3
    (7, 27, 96, 150, 3, 2, 1, "C=16> units=800 of 16 waves=4"),
    (6, 27, 96, 150, 3, 2, 1, "C=4> units=1311 of 8 waves=4")])
def test_waves_of_a_tiled_unit(n, h, c, oc, k, abits, wbits, plan):
    d = bs.bs_conv2d_describe(conv(n, h, h, c, oc, k, 1, abits, wbits, U, B))
    assert d.startswith("conv_generic_kernel_tiled"), d
    got = re.search(r"(C=\d+>).* (units=\d+ of \d+) channels "
                    r"waves_per_unit=(\d)", d)
    assert "%s %s waves=%s" % got.groups() == plan, d


@pytest.mark.parametrize("m,k,n,abits,wbits,rows", [
    # waves per SIMD of 4 rows x 4 columns (A W <= 4) or of one row, against
    # the pixel kernel: 3 (8 of one row), any up to 8 (10) rows
    (16, 1024, 3072, 2, 2, True), (16, 1024, 3076, 2, 2, False),
    (8, 1024, 65536, 2, 2, True), (11, 1024, 4096, 4, 4, False),
    (10, 1024, 65536, 4, 4, True), (16, 2048, 65536, 2, 2, True),
    # one bit a pair: 2 and 4 from 5 rows on, 24 and 12
    (8, 1024, 4096, 1, 1, True), (8, 1024, 4100, 1, 1, False),
    (4, 1024, 65536, 1, 1, True), (16, 2048, 4096, 1, 1, True),
    (16, 2048, 4100, 1, 1, False), (32, 4096, 6144, 1, 1, True),
    (32, 4096, 6148, 1, 1, False), (24, 4096, 16384, 1, 1, True),
    (24, 4096, 16388, 1, 1, False), (16, 4096, 65536, 1, 1, True),
    # 32 rows: 32 and 64
    (32, 4096, 16384, 2, 2, True), (32, 4096, 16388, 2, 2, False),
    (32, 4096, 4096, 4, 4, True), (32, 4096, 8192, 4, 4, True),
    (32, 4096, 8196, 4, 4, False), (24, 4096, 65536, 4, 4, True),
    # against the tiled kernel: 2, 8 or 6, 6 and 20
    (16, 768, 2048, 2, 2, True), (16, 768, 2052, 2, 2, False),
    (16, 768, 2048, 4, 4, True), (16, 768, 2052, 4, 4, False),
    (16, 1024, 1536, 8, 8, True), (16, 1024, 1540, 8, 8, False),
    (32, 3072, 3072, 2, 1, True), (32, 3072, 3076, 2, 1, False),
    (16, 768, 50000, 4, 4, False), (32, 4096, 2560, 8, 8, True),
    (32, 4096, 2564, 8, 8, False),
    # one row: 8, 64
    (1, 768, 32768, 2, 2, True), (1, 768, 32772, 2, 2, False),
    (1, 4096, 65536, 2, 2, True),
    # rows and words as before
    (17, 1024, 64, 2, 2, False), (16, 704, 64, 2, 2, False)])
def test_few_rows(m, k, n, abits, wbits, rows):
    assert (family(dense(m, k, n, abits, wbits)) == "dense_rows") == rows


@pytest.mark.parametrize("p,tiled", [
    # few units of 64 pixels x 4 channels
    (conv(1, 7, 7, 512, 512, 3, 1, 1, 1), True),          # 128
    (conv(4, 7, 7, 512, 512, 3, 1, 1, 1), False),         # 512
    (conv(4, 7, 7, 512, 512, 3, 1, 1, 1, U, B), True),
    (conv(6, 7, 7, 512, 512, 3, 1, 1, 1, U, B), False),   # 640
    (conv(6, 7, 7, 512, 512, 3, 1, 2, 1), True),          # 640
    (conv(8, 7, 7, 512, 512, 3, 1, 2, 1), False),         # 896
    (conv(1, 14, 14, 512, 512, 1, 1, 2, 2), False),       # 16 words
    (dense(256, 4096, 512, 1, 1), True),                  # 512, products
    (dense(320, 4096, 512, 1, 1), False),                 # 640
    (dense(256, 4096, 512, 2, 1), False),                 # 512
    (dense(256, 4096, 256, 2, 1), True),                  # 256
    (dense(256, 1024, 512, 2, 1), True),                  # 512, 32 words
    (dense(256, 4096, 512, 2, 2), True),
    (dense(320, 4096, 512, 2, 2), False),                 # 640
    (dense(320, 4096, 512, 4, 4), True),
    # one unit per wave in a full round
    (conv(64, 7, 7, 512, 512, 3, 1, 2, 1), True),
    (conv(32, 14, 14, 256, 256, 3, 1, 2, 1), False),      # 8 words
    (conv(64, 14, 14, 256, 256, 3, 2, 2, 1), True),
    (conv(64, 7, 7, 512, 512, 3, 1, 3, 1), False),        # 24.5 units per CU
    (conv(40, 7, 7, 512, 512, 3, 1, 3, 1), True),         # 15.5
    (dense(1792, 1024, 1024, 2, 1), True),
    (conv(16, 28, 28, 512, 128, 1, 1, 3, 1), False)])     # 16 words
def test_long_reductions(p, tiled):
    assert family(p) == ("conv_generic" if tiled else "conv_pix")
    assert ("tiled" in bs.bs_conv2d_describe(p)) == tiled


@pytest.mark.parametrize("p,kernel", [
    # 2 and 4 words per plane: channels on lanes
    (dense(1900, 64, 66, 2, 1, U, B), "conv_ocl_kernel"),
    (dense(32768, 64, 66, 2, 1, U, B), "conv_ocl_kernel"),    # 16 Ki lanes a CU
    (dense(32770, 64, 66, 2, 1, U, B), "conv_generic_kernel_tiled"),
    (dense(16384, 64, 10, 2, 1, U, B), "conv_ocl_kernel"),
    (dense(16388, 64, 10, 2, 1, U, B), "conv_generic_kernel_tiled"),
    (dense(9362, 64, 849, 2, 1, U, B), "conv_ocl_kernel"),    # 32 Ki
    (dense(9364, 64, 849, 2, 1, U, B), "conv_generic_kernel_tiled"),
    (dense(15000, 64, 402, 4, 4, U, B), "conv_ocl_kernel"),
    (dense(15000, 64, 402, 2, 2, U, B), "conv_generic_kernel_tiled"),
    (dense(1900, 64, 66, 4, 4, U, B), "conv_generic_kernel_tiled"),
    (dense(1900, 128, 66, 2, 1, U, B), "conv_ocl_kernel"),
    (dense(1900, 192, 66, 2, 1, U, B), "conv_generic_kernel_tiled"),
    # one word: one output per thread, up to 192 Ki or 128 Ki outputs
    (dense(3072, 32, 64, 2, 2, S, U), "conv_generic_kernel A"),
    (dense(3073, 32, 64, 2, 2, S, U), "conv_generic_kernel_tiled"),
    (dense(2048, 32, 64, 4, 4, S, U), "conv_generic_kernel A"),
    (dense(2049, 32, 64, 4, 4, S, U), "conv_generic_kernel_tiled"),
    (dense(64, 32, 64, 4, 8, S, U), "conv_generic_kernel_tiled"),
    (dense(64, 32, 64, 8, 7, S, U), "conv_generic_kernel A"),
    (dense(64, 64, 64, 2, 2, S, U), "conv_generic_kernel_tiled")])
def test_short_reductions(p, kernel):
    assert bs.bs_conv2d_describe(p).startswith(kernel)


def test_run_length_keeps_the_pixel_kernel():
    """A run length set for the pixels-on-lanes kernel is used in mode 0 on
    every shape that has one."""
    for p in (conv(1, 7, 7, 512, 512, 3, 1, 2, 1), dense(256, 4096, 256, 2, 2),
              dense(16, 1024, 512, 2, 2), conv(64, 7, 7, 512, 512, 3, 1, 2, 1)):
        assert family(p) != "conv_pix"
        bs.bs_set_units_per_wave(3)
        d = bs.bs_conv2d_describe(p)
        assert d.startswith("conv_pix_kernel") and "units_per_wave=3" in d
        bs.bs_set_units_per_wave(0)
    # none here: the call keeps its kernel
    for p in (dense(16, 800, 64, 2, 2), conv(1, 9, 9, 96, 10, 3, 1, 2, 1)):
        before = bs.bs_conv2d_describe(p)
        bs.bs_set_units_per_wave(3)
        assert bs.bs_conv2d_describe(p) == before
        bs.bs_set_units_per_wave(0)
