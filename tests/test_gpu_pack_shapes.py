"""GPU parity of the pack kernels at the edges of their tiles, against the
oracle: rows whose length is no multiple of 32 (chunks of 64 elements, eight
to a wave, running over row ends), and strided reduction axes (groups of four
rows with overlapping last groups, tiles that span outer indices, one to
eight and more words per plane, all three layouts), at 1-8 bits."""
import numpy as np
import pytest
import torch

from paper_1810_11066_amd import bitserial as bs

pytestmark = pytest.mark.gpu

SENT32 = 0x7FFFFFFF
GUARD = 1024


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU parity tests need the MI355X"
    bs.load_library()


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

    def words(self):
        torch.cuda.synchronize()
        b = self.buf.cpu()
        assert bool((b[:GUARD] == SENT32).all()), "write before output"
        assert bool((b[GUARD + self.n:] == SENT32).all()), "write past output"
        return b[GUARD:GUARD + self.n].numpy().view(np.uint32)


# k: below, at and above chunk and word ends; rows: fewer and more chunks than
# a wave takes, and a grid that strides
ROWS = [(1, 1), (3, 31), (7, 33), (9, 63), (17, 65), (5, 100), (33, 127),
        (8, 129), (2, 1000), (1, 4097), (70000, 45), (300000, 5)]


@pytest.mark.parametrize("rows,k", ROWS)
@pytest.mark.parametrize("bits", [1, 3, 8])
def test_pack_any_k(oracle, rows, k, bits):
    rng = np.random.default_rng(rows * 7 + k)
    q = rng.integers(0, 256, size=(rows, k), dtype=np.uint8)
    say("pack", rows, k, bits)
    want = oracle.pack(q, bits)
    g = Guarded(want.size)
    bs.bs_pack(dev(q), g.t, rows, k, bits)
    assert np.array_equal(g.words().reshape(want.shape), want)


@pytest.mark.parametrize("rows,k", ROWS)
@pytest.mark.parametrize("enc,bits", [(bs.UNIPOLAR, 2), (bs.BIPOLAR, 1),
                                      (bs.SIGNED, 4)])
def test_quantize_pack_any_k(oracle, rows, k, enc, bits):
    rng = np.random.default_rng(rows + 11 * k + enc)
    x = rng.standard_normal((rows, k), dtype=np.float32) * 4
    special = np.array([np.nan, np.inf, -np.inf, -0.0, 0.0, 1e-42, 0.5, 1.5],
                       dtype=np.float32)
    x.reshape(-1)[:: max(1, x.size // 64)] = np.resize(
        special, x.reshape(-1)[:: max(1, x.size // 64)].size)
    say("quantize_pack", rows, k, enc, bits)
    want = oracle.pack(oracle.quantize(x, 0.9, bits, enc), bits)
    g = Guarded(want.size)
    bs.bs_quantize_pack(dev(x), g.t, rows, k, 0.9, bits, enc)
    assert np.array_equal(g.words().reshape(want.shape), want)


# outer, k, inner
STRIDED = [(1, 1, 2), (3, 40, 3), (2, 32, 4), (5, 33, 5), (70, 64, 9),
           (2, 100, 49), (1, 260, 1027), (3, 256, 196), (40, 96, 25),
           (1, 31, 4099), (300, 70, 7), (600, 129, 1), (2, 513, 130)]


@pytest.mark.parametrize("shape", STRIDED, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("bits", [1, 3, 8])
def test_pack_strided(oracle, shape, layout, bits):
    outer, k, inner = shape
    rng = np.random.default_rng(outer + 3 * k + 5 * inner)
    q = rng.integers(0, 256, size=shape, dtype=np.uint8)
    say("pack_ex", shape, layout, bits)
    want = oracle.pack_ex(q, bits, axis=1, layout=layout)
    g = Guarded(want.size)
    bs.bs_pack_ex(dev(q), g.t, outer, k, inner, bits, layout)
    assert np.array_equal(g.words().reshape(want.shape), want)


@pytest.mark.parametrize("bits", range(1, 9))
def test_quantize_halves(oracle, bits):
    """Every value half way between two codes, its float32 neighbours, the
    ends of the range and the special values, through each unipolar
    quantizer: round half to even, then clamp."""
    h = np.arange(-4, 2 * (1 << bits) + 4, dtype=np.float32) / 2
    x = np.concatenate([h, np.nextafter(h, np.float32(np.inf)),
                        np.nextafter(h, np.float32(-np.inf)),
                        np.array([np.nan, np.inf, -np.inf, -0.0, 1e-42, -1e-42,
                                  3e38, -3e38], dtype=np.float32)])
    x = np.resize(x, (x.size + 63) // 64 * 64).astype(np.float32)
    say("halves", bits, x.size)
    want = oracle.quantize(x, 1.0, bits)
    q = torch.empty(x.size, dtype=torch.uint8, device="cuda")
    bs.bs_quantize(dev(x), q, 1.0, bits)
    assert np.array_equal(q.cpu().numpy(), want)
    for k in (64, 8):
        g = Guarded(x.size // k * bits * ((k + 31) // 32))
        bs.bs_quantize_pack(dev(x), g.t, x.size // k, k, 1.0, bits)
        wp = oracle.pack(want.reshape(-1, k), bits)
        assert np.array_equal(g.words().reshape(wp.shape), wp)


def test_more_than_2_31_chunks():
    """Row numbers past 32 bits: 2^31 + 100 rows of one code (each row one
    chunk) pack to their own low bit."""
    rows = 2 ** 31 + 100
    q = torch.randint(0, 256, (rows,), dtype=torch.uint8, device="cuda")
    out = torch.full((rows,), SENT32, dtype=torch.int32, device="cuda")
    say("pack", rows, 1)
    bs.bs_pack(q, out, rows, 1, 1)
    torch.cuda.synchronize()
    for a in range(0, rows, 1 << 28):
        b = min(rows, a + (1 << 28))
        assert torch.equal(out[a:b], (q[a:b] & 1).int())
    # and with a stride of 2: each row one group of a tile
    out.fill_(SENT32)
    say("pack_ex", rows // 2, 1, 2)
    bs.bs_pack_ex(q, out, rows // 2, 1, 2, 1, bs.LAYOUT_BMK)
    torch.cuda.synchronize()
    for a in range(0, rows, 1 << 28):
        b = min(rows, a + (1 << 28))
        assert torch.equal(out[a:b], (q[a:b] & 1).int())


@pytest.mark.parametrize("rows,k", [(2048, 165), (6144, 33), (6145, 33),
                                    (3000, 70)])
@pytest.mark.parametrize("bits", [1, 4, 8])
def test_chunks_per_wave(oracle, rows, k, bits):
    """Up to 6144 chunks a wave takes one, above it eight: codes and floats on
    both sides."""
    rng = np.random.default_rng(rows + k)
    q = rng.integers(0, 256, size=(rows, k), dtype=np.uint8)
    say("pack", rows, k, bits)
    want = oracle.pack(q, bits)
    g = Guarded(want.size)
    bs.bs_pack(dev(q), g.t, rows, k, bits)
    assert np.array_equal(g.words().reshape(want.shape), want)
    x = rng.standard_normal((rows, k), dtype=np.float32) * 100
    for enc in (bs.UNIPOLAR, bs.BIPOLAR if bits == 1 else bs.SIGNED):
        say("quantize_pack", rows, k, enc, bits)
        want = oracle.pack(oracle.quantize(x, 0.7, bits, enc), bits)
        g = Guarded(want.size)
        bs.bs_quantize_pack(dev(x), g.t, rows, k, 0.7, bits, enc)
        assert np.array_equal(g.words().reshape(want.shape), want)


# one and four rows to a thread (128 workgroups of four), one word per plane
# and row stored without LDS, tiles of up to 64 words along contiguous codes
@pytest.mark.parametrize("shape", [
    (127, 256, 128), (128, 256, 128), (130, 250, 129), (64, 3, 12544),
    (9, 3, 1001), (2000, 31, 17), (64, 4096, 1), (50, 2070, 1), (700, 64, 1),
    (33, 1000, 1)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("bits", [1, 3, 8])
def test_pack_strided_tiles(oracle, shape, layout, bits):
    outer, k, inner = shape
    rng = np.random.default_rng(outer + k + inner)
    q = rng.integers(0, 256, size=shape, dtype=np.uint8)
    say("pack_ex", shape, layout, bits)
    want = oracle.pack_ex(q, bits, axis=1, layout=layout)
    g = Guarded(want.size)
    bs.bs_pack_ex(dev(q), g.t, outer, k, inner, bits, layout)
    assert np.array_equal(g.words().reshape(want.shape), want)
