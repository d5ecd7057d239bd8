"""GPU parity of both kernels of every pixels-on-lanes specialisation -- the one
for lone waves and the one for several waves per SIMD -- against the plain
kernel (kernel mode 1), on packed activations, codes, float32 values, with
requantized output and paired.  The run length decides which one a grid takes:
260 workgroups or more, or at most 256."""
import pytest
import torch

from paper_1810_11066_amd import bitserial as bs

pytestmark = pytest.mark.gpu

U, B, S = bs.UNIPOLAR, bs.BIPOLAR, bs.SIGNED
OC = 64


@pytest.fixture(autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU parity tests need the MI355X"
    bs.load_library()
    yield
    bs.bs_set_kernel_mode(0)
    bs.bs_set_units_per_wave(0)


def say(*a):
    print(*a, flush=True)


def codes(shape, bits, gen):
    return torch.randint(0, 1 << bits, shape, dtype=torch.uint8, device="cuda",
                         generator=gen)


def both(call, numel, described=None):
    """call(out) with several waves per SIMD, with lone waves, and by the
    plain kernel: the same words."""
    outs = []
    for mode, run in ((0, 1), (0, 8), (1, 0)):
        bs.bs_set_kernel_mode(3 if mode == 0 else 1)
        bs.bs_set_units_per_wave(run)
        if described is not None and mode == 0:
            d = described()
            assert d.startswith("conv_pix_kernel"), d
            assert d.endswith(" lone waves") == (run == 8), d
        outs.append(torch.full((numel,), -7, dtype=torch.int32, device="cuda"))
        call(outs[-1])
    bs.bs_set_kernel_mode(0)
    bs.bs_set_units_per_wave(0)
    assert torch.equal(outs[0], outs[2]), "several waves per SIMD"
    assert torch.equal(outs[1], outs[2]), "lone waves"


CASES = ([(a, w, U, U) for a in range(1, 5) for w in range(1, 5)] +
         [(a, 1, U, B) for a in range(1, 5)] +
         [(a, w, U, S) for a in range(1, 5) for w in range(2, 5)] +
         [(a, a, S, S) for a in range(2, 5)] + [(1, 1, B, U), (1, 1, B, B)])


@pytest.mark.parametrize("bits", CASES, ids=lambda b: "A%d%sW%d%s" % (
    b[0], "ubs"[b[2]], b[1], "ubs"[b[3]]))
def test_both_kernels(bits):
    abits, wbits, aenc, wenc = bits
    gen = torch.Generator("cuda").manual_seed(abits * 10 + wbits)
    staged = aenc == U and wenc != S
    for k, s, cw in [(k, s, 1 << e) for k in (1, 3) for s in (1, 2)
                     for e in range(8 if k == 1 else 5)]:
        h, w = (13, 16) if s == 1 else (25, 31)
        n, c = 40, 32 * cw                 # 130 groups of 64 output pixels
        p = bs.ConvParams(n, h, w, c, OC, k, k, s, s, k // 2, k // 2, *bits)
        bs.bs_set_kernel_mode(3)
        if not bs.bs_conv2d_describe(p).startswith("conv_pix_kernel"):
            bs.bs_set_kernel_mode(0)
            continue                       # no specialisation
        say("both kernels", bits, k, s, c)
        oh, ow = bs.bs_conv2d_out_shape(p)
        numel = n * oh * ow * OC
        x = codes((n, h, w, c), abits, gen)
        a = bs.pack(x, abits)
        wq = bs.pack(codes((OC, k, k, c), wbits, gen), wbits)
        # 9 to 18 word pairs a result are served by one kernel in any grid
        pairs = k * k * cw * abits * wbits
        both(lambda o: bs.bs_conv2d(p, a, wq, o), numel,
             None if pairs <= 9 and abits <= 3 or aenc == wenc == B
             else lambda: bs.bs_conv2d_describe(p))
        if not staged:
            continue
        want = torch.empty(numel, dtype=torch.int32, device="cuda")
        bs.bs_set_kernel_mode(1)
        bs.bs_conv2d(p, a, wq, want)
        bs.bs_set_kernel_mode(0)
        for run in (1, 4):
            bs.bs_set_units_per_wave(run)
            got = torch.full_like(want, -7)
            try:
                bs.bs_conv2d_codes(p, x, wq, got)
            except bs.BitserialError as e:
                assert e.status == bs.BS_ERR_UNSUPPORTED
            else:
                assert torch.equal(got, want), "codes"
            if k == 1:
                got.fill_(-7)
                try:
                    bs.bs_conv2d_quantized(p, x.float(), 1.0, wq, got)
                except bs.BitserialError as e:
                    assert e.status == bs.BS_ERR_UNSUPPORTED
                else:
                    assert torch.equal(got, want), "quantized"
        bs.bs_set_units_per_wave(0)
        scale = 7.0 / float(want.abs().float().mean() * 2 + 1)
        words = n * oh * ow * 3 * bs.words(OC)
        both(lambda o: bs.bs_conv2d_requant(p, a, wq, scale, 3, o), words)
        if k == 3:
            w1 = bs.pack(codes((OC, 1, 1, c), wbits, gen), wbits)

            def pair(o):
                bs.bs_conv2d_pair(p, a, wq, w1, o[:numel], o[numel:])
            both(pair, 2 * numel)

            def pair_requant(o):
                bs.bs_conv2d_pair_requant(p, a, wq, w1, scale, 4 * scale, 3,
                                          o[:words], o[words:])
            both(pair_requant, 2 * words)
