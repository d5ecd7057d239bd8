"""GPU parity of conv_generic_kernel_tiled, the run-time-shaped kernel of the
shapes no specialisation covers, against the oracle: every group of planes
(1-8 bits), chunk width (1-4 words, whole and partial last chunks), channel
tile and remainder, window, stride and padding, the encodings' corrections,
waves that share a unit's steps, operands swapped for products of few rows,
and requantized output; and of dense_rows_kernel, which serves products of few
rows and many words."""
import numpy as np
import pytest
import torch

from paper_1810_11066_amd import bitserial as bs

pytestmark = pytest.mark.gpu

SENT32 = 0x7FFFFFFF
GUARD = 1024
U, B, S = bs.UNIPOLAR, bs.BIPOLAR, bs.SIGNED


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU parity tests need the MI355X"
    bs.load_library()
    bs.bs_set_kernel_mode(0)
    yield
    bs.bs_set_kernel_mode(0)


def say(*a):
    print(*a, flush=True)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Guarded:
    def __init__(self, numel):
        self.n = numel
        self.buf = torch.full((numel + 2 * GUARD,), SENT32, dtype=torch.int32,
                              device="cuda")
        self.t = self.buf[GUARD:GUARD + numel]

    def numpy(self):
        torch.cuda.synchronize()
        b = self.buf.cpu()
        assert bool((b[:GUARD] == SENT32).all()), "write before output"
        assert bool((b[GUARD + self.n:] == SENT32).all()), "write past output"
        return b[GUARD:GUARD + self.n].numpy()


def operands(oracle, seed, n, h, w, c, oc, kh, kw, s, pad, abits, wbits, aenc,
             wenc):
    rng = np.random.default_rng(seed)
    a = rng.integers(0, 1 << abits, size=(n, h, w, c), dtype=np.uint8)
    wq = rng.integers(0, 1 << wbits, size=(oc, kh, kw, c), dtype=np.uint8)
    ap, wp = oracle.pack(a, abits), oracle.pack(wq, wbits)
    want = oracle.conv2d(oracle.conv_params(n, h, w, c, oc, kh, kw, s, pad,
                                            abits, wbits, aenc, wenc), ap, wp)
    p = bs.ConvParams(n, h, w, c, oc, kh, kw, s[0], s[1], pad[0], pad[1],
                      abits, wbits, aenc, wenc)
    return ap, wp, want, p


def run_conv(oracle, seed, *shape):
    say("tiled conv", shape)
    ap, wp, want, p = operands(oracle, seed, *shape)
    assert bs.bs_conv2d_describe(p).startswith("conv_generic_kernel_tiled")
    g = Guarded(want.size)
    bs.bs_conv2d(p, dev(ap.view(np.int32)), dev(wp.view(np.int32)), g.t)
    assert np.array_equal(g.numpy().reshape(want.shape), want)


SHAPES = [
    # n, h, w, c, oc, (kh, kw), (sh, sw), (ph, pw)
    (2, 7, 9, 90, 24, (3, 3), (1, 1), (1, 1)),     # 3 words, whole chunks
    (1, 9, 7, 130, 13, (3, 3), (2, 2), (1, 1)),    # 5 words: 3 + 2
    (1, 6, 8, 200, 30, (3, 3), (1, 1), (2, 2)),    # 7 words: 4 + 3
    (1, 11, 5, 64, 18, (5, 5), (1, 1), (2, 2)),    # 2 words
    (3, 5, 13, 17, 6, (3, 3), (1, 1), (1, 1)),     # 1 word
    (1, 12, 10, 128, 20, (2, 5), (3, 1), (0, 3)),  # window, stride, pad differ
    (1, 4, 4, 96, 3, (7, 7), (1, 1), (3, 3)),      # window past the image
    (1, 9, 9, 352, 33, (1, 1), (1, 1), (0, 0)),    # one tap, 11 words
    (2, 8, 8, 64, 7, (1, 1), (2, 2), (1, 1)),      # pad 1 around 1x1 windows
]
BITS = [(1, 1, U, U), (2, 1, U, B), (1, 2, B, U), (1, 1, B, B), (2, 2, S, U),
        (2, 3, U, S), (3, 3, S, S), (4, 1, U, U), (1, 4, U, B), (4, 2, B, S),
        (4, 4, B, B), (5, 3, U, U), (8, 1, S, B), (2, 7, U, S), (6, 6, S, B),
        (1, 1, B, U), (1, 3, B, S), (1, 4, B, B), (1, 7, B, S)]


@pytest.mark.parametrize("bits", BITS, ids=lambda b: "A%d%sW%d%s" % (
    b[0], "ubs"[b[2]], b[1], "ubs"[b[3]]))
def test_conv_encodings(oracle, bits):
    """Every shape at one choice of widths and encodings."""
    abits, wbits, aenc, wenc = bits
    for i, (n, h, w, c, oc, k, s, pad) in enumerate(SHAPES):
        spec = bs.ConvParams(n, h, w, c, oc, *k, *s, *pad, *bits)
        if not bs.bs_conv2d_describe(spec).startswith("conv_generic"):
            continue        # served by a specialised kernel
        run_conv(oracle, 100 * i + abits * 9 + wbits, n, h, w, c, oc, *k, s,
                 pad, *bits)


@pytest.mark.parametrize("npix,oc", [
    (64, 4), (65, 5), (130, 12), (63, 16), (64, 17), (200, 31), (128, 150),
    (4100, 150), (20000, 40)])
def test_conv_tiles(oracle, npix, oc):
    """Pixel groups and channel tiles at their edges, in the 4-channel tiles
    that these grids take, from one unit whose steps are shared to thousands
    of units (test_wide_tiles has the wider ones)."""
    for abits, wbits in ((1, 1), (2, 2), (3, 3)):
        if npix * oc > 10 ** 5 and abits > 1:
            continue
        run_conv(oracle, npix + oc, 1, 1, npix, 96, oc, 1, 3, (1, 1), (0, 1),
                 abits, wbits, U, U)


@pytest.mark.parametrize("m", [1, 2, 5, 16, 18, 32, 47, 63, 64])
@pytest.mark.parametrize("n,k", [(1, 40), (70, 100), (129, 800), (1000, 352),
                                 (3, 768), (34, 2080), (6, 4150)])
def test_dense_few_rows(oracle, m, n, k):
    """Matrix products of few rows over the encodings: the reduction on the
    lanes (from 24 words per plane, whole and partial chunks of 64 words, row
    and channel tiles with remainders), and pixels or output channels on
    them."""
    for abits, wbits, aenc, wenc in ((1, 1, U, U), (2, 2, U, S), (1, 3, B, U),
                                     (2, 1, U, B), (1, 1, B, B), (4, 4, S, S),
                                     (4, 2, B, B), (6, 5, S, B)):
        say("dense", m, n, k, abits, wbits, aenc, wenc)
        rng = np.random.default_rng(m * 1000 + n + k)
        a = rng.integers(0, 1 << abits, size=(m, k), dtype=np.uint8)
        wq = rng.integers(0, 1 << wbits, size=(n, k), dtype=np.uint8)
        ap, wp = oracle.pack(a, abits), oracle.pack(wq, wbits)
        op = oracle.conv_params(1, 1, m, k, n, 1, 1, 1, 0, abits, wbits, aenc,
                                wenc)
        want = oracle.conv2d(op, ap.reshape(1, 1, m, abits, -1),
                             wp.reshape(n, 1, 1, wbits, -1)).reshape(m, n)
        rows = (m <= 16 and k > 23 * 32) or (m <= 32 and k > 95 * 32)
        p = bs.ConvParams(1, 1, m, k, n, 1, 1, 1, 1, 0, 0, abits, wbits, aenc,
                          wenc)
        assert bs.bs_conv2d_describe(p).startswith(
            "dense_rows_kernel") == rows
        g = Guarded(m * n)
        bs.bs_dense_ex(m, n, k, abits, aenc, wbits, wenc,
                       dev(ap.view(np.int32)), dev(wp.view(np.int32)), g.t)
        assert np.array_equal(g.numpy().reshape(m, n), want)


@pytest.mark.parametrize("shape,abits,wbits,tiled", [
    # n, h, w, c, oc, k, s: long reductions with few units of 64 pixels x 4
    # channels (at most 768), and above
    ((1, 7, 7, 512, 64, 3, 1), 2, 1, True),
    ((2, 9, 9, 512, 1020, 3, 1), 3, 3, True),
    ((2, 9, 9, 512, 1028, 3, 1), 3, 3, False),
    ((1, 1, 200, 4096, 64, 1, 1), 2, 2, True),
    # one unit per wave in a full round (3072 to 7168 units), A >= 2, W = 1
    ((4, 7, 7, 512, 3068, 3, 1), 2, 1, False),
    ((4, 7, 7, 512, 3072, 3, 1), 2, 1, True),
    ((4, 7, 7, 512, 3072, 3, 1), 1, 1, False),
    ((1, 1, 64 * 28, 1024, 1024, 1, 1), 2, 1, True),
    ((1, 1, 64 * 28 + 1, 1024, 1024, 1, 1), 2, 1, False)])
def test_rule_for_long_reductions(oracle, shape, abits, wbits, tiled):
    """The kernel on each side of the lines, and its results."""
    n, h, w, c, oc, k, s = shape
    say("long reduction", shape, abits, wbits)
    ap, wp, want, p = operands(oracle, c + oc, n, h, w, c, oc, k, k, (s, s),
                               (k // 2, k // 2), abits, wbits, U, U)
    assert bs.bs_conv2d_describe(p).startswith(
        "conv_generic_kernel_tiled" if tiled else "conv_pix_kernel")
    g = Guarded(want.size)
    bs.bs_conv2d(p, dev(ap.view(np.int32)), dev(wp.view(np.int32)), g.t)
    assert np.array_equal(g.numpy().reshape(want.shape), want)


@pytest.mark.parametrize("oc", [3, 8, 21, 40, 150])
@pytest.mark.parametrize("obits", [1, 3, 8])
def test_requant(oracle, oc, obits):
    for i, (abits, wbits, aenc, wenc) in enumerate(
            ((2, 1, U, U), (3, 3, S, S), (1, 1, B, B), (4, 4, U, U))):
        shape = (2, 9, 7, 96, oc, 3, 3, (1, 1), (1, 1), abits, wbits, aenc,
                 wenc)
        say("tiled requant", shape, obits)
        ap, wp, conv, p = operands(oracle, 7 * oc + i, *shape)
        scale = ((1 << obits) - 1) / max(1.0, float(abs(conv).max()))
        want = oracle.pack(oracle.quantize(conv.astype(np.float32), scale,
                                           obits), obits)
        g = Guarded(want.size)
        bs.bs_conv2d_requant(p, dev(ap.view(np.int32)),
                             dev(wp.view(np.int32)), scale, obits, g.t)
        got = g.numpy().view(np.uint32)
        assert np.array_equal(got.reshape(want.shape), want)


# n, h, w, c, oc, (kh, kw), abits, wbits, aenc, wenc, channels per tile: grids of
# more than four waves a SIMD, units of 16 channels with a ragged last one
WIDE = [
    (48, 27, 27, 96, 150, (3, 3), 2, 1, U, B, 16),     # chunks of 3 words
    (48, 27, 27, 17, 150, (3, 3), 1, 2, U, S, 16),     # 1 word
    (48, 27, 27, 64, 150, (5, 5), 2, 2, S, U, 16),     # 2 words
    (96, 27, 27, 130, 78, (3, 3), 1, 4, U, U, 16),     # 3 + 2 words
    (48, 27, 27, 200, 150, (1, 3), 4, 1, U, U, 16),    # 4 + 3 words
    (48, 27, 27, 96, 150, (3, 3), 2, 1, B, U, 16),     # SW pass
    (48, 27, 27, 96, 150, (3, 3), 1, 2, B, B, 16),     # +-1 activations
    (48, 27, 27, 70, 152, (3, 3), 1, 1, B, B, 16),     # XNOR, whole quads
    (48, 27, 27, 96, 158, (3, 3), 2, 3, U, U, 8),
    (48, 27, 27, 60, 158, (3, 3), 4, 2, B, S, 8),      # SW pass
    (48, 27, 27, 96, 158, (2, 3), 5, 2, S, U, 8),      # 3 + 2 planes
    (48, 27, 27, 96, 158, (3, 3), 3, 3, U, B, 4),      # four tiles to a unit
    (48, 27, 27, 40, 160, (3, 1), 6, 5, B, B, 4),      # plane groups, SW passes
]


def wide(shape):
    n, h, w, c, oc, (kh, kw), abits, wbits, aenc, wenc, _ = shape
    say("wide tiles", shape)
    p = bs.ConvParams(n, h, w, c, oc, kh, kw, 1, 1, kh // 2, kw // 2, abits,
                      wbits, aenc, wenc)
    gen = torch.Generator("cuda").manual_seed(c + oc + abits)
    a = bs.pack(torch.randint(0, 1 << abits, (n, h, w, c), dtype=torch.uint8,
                              device="cuda", generator=gen), abits)
    wq = bs.pack(torch.randint(0, 1 << wbits, (oc, kh, kw, c),
                               dtype=torch.uint8, device="cuda",
                               generator=gen), wbits)
    return p, a, wq


def plain(call):
    bs.bs_set_kernel_mode(1)
    try:
        call()
    finally:
        bs.bs_set_kernel_mode(0)


@pytest.mark.parametrize("shape", WIDE, ids=lambda s: "C%d_A%d%sW%d%s" % (
    s[10], s[6], "ubs"[s[8]], s[7], "ubs"[s[9]]))
def test_wide_tiles(shape):
    """The channel tiles of grids that fill the chip, int32 and requantized,
    against the plain kernel."""
    p, a, wq = wide(shape)
    d = bs.bs_conv2d_describe(p)
    assert d.startswith("conv_generic_kernel_tiled") and " of 16 channels " in d
    assert ",C=%d" % shape[10] in d, d
    oh, ow = bs.bs_conv2d_out_shape(p)
    numel = p.n * oh * ow * p.oc
    want = torch.empty(numel, dtype=torch.int32, device="cuda")
    plain(lambda: bs.bs_conv2d(p, a, wq, want))
    g = Guarded(numel)
    bs.bs_conv2d(p, a, wq, g.t)
    g.numpy()
    assert torch.equal(g.t, want)
    scale = 7.0 / float(want.abs().float().mean() * 2 + 1)
    words = p.n * oh * ow * 3 * bs.words(p.oc)
    want = torch.empty(words, dtype=torch.int32, device="cuda")
    plain(lambda: bs.bs_conv2d_requant(p, a, wq, scale, 3, want))
    g = Guarded(words)
    bs.bs_conv2d_requant(p, a, wq, scale, 3, g.t)
    g.numpy()
    assert torch.equal(g.t, want)


def test_batch_split():
    """An int32 output past 2 GiB, and packed activations past it with
    requantized output: several launches of the tiled kernel."""
    p, a, wq = wide((130, 56, 56, 32, 1342, (1, 1), 1, 1, U, U, 16))
    d = bs.bs_conv2d_describe(p)
    assert d.startswith("conv_generic_kernel_tiled") and "batch split" in d
    numel = 130 * 56 * 56 * 1342
    want = torch.empty(numel, dtype=torch.int32, device="cuda")
    plain(lambda: bs.bs_conv2d(p, a, wq, want))
    g = Guarded(numel)
    bs.bs_conv2d(p, a, wq, g.t)
    torch.cuda.synchronize()
    assert torch.equal(g.t, want)
    assert bool((g.buf[:GUARD] == SENT32).all())
    assert bool((g.buf[-GUARD:] == SENT32).all())
    del g, want
    # 7200 x 56 x 56 pixels of 96 bytes
    n = 7200
    p = bs.ConvParams(n, 56, 56, 96, 10, 1, 1, 1, 1, 0, 0, 8, 1, U, U)
    a = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, 56, 56, 8, 3),
                      dtype=torch.int32, device="cuda")
    wq = bs.pack(torch.randint(0, 2, (10, 1, 1, 96), dtype=torch.uint8,
                               device="cuda"), 1)
    say("batch split, requantized", n)
    words = n * 56 * 56 * 2
    want = torch.empty(words, dtype=torch.int32, device="cuda")
    plain(lambda: bs.bs_conv2d_requant(p, a, wq, 3e-4, 2, want))
    got = torch.full((words,), SENT32, dtype=torch.int32, device="cuda")
    bs.bs_conv2d_requant(p, a, wq, 3e-4, 2, got)
    assert torch.equal(got, want)
