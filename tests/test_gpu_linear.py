"""GPU tests: linear layers of 4-bit codes against whole-number sums in fp64."""
import pytest

torch = pytest.importorskip("torch")


# Every cut (tokens / waves / steps of a unit) with and without a padded unit, blocks of channels that are not whole, the longest K
# that fits and the next, large layers of K a multiple of 192; -8 among the codes.  The sums are whole numbers below 2^24: the integer
# result is equal, fp32 results are a few roundings (the scales, 4; with the planes' weights and sums, 8) from the exact value, fp16
# results half an ulp more.  (The planes take the same cuts by their own costs.)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n,cut", [
    (1, 64, 1, "64/4/2"), (33, 64, 40, "64/4/2"), (31, 128, 8, "64/4/2"), (130, 320, 333, "32/4/5"), (1000, 640, 96, "32/4/5"),
    (2100, 448, 1000, "64/8/4"), (9000, 704, 640, "128/8/4"), (70000, 64, 72, "128/4/2"), (4300, 768, 1160, "128/8/4"),
    (40, 6400, 33, "tile"), (40, 6784, 33, "tile"), (700, 2560, 264, "32/4/8"), (20, 8192, 40, "tile"),
    (40, 6080, 33, "32/4/8"), (40, 6208, 33, "tile"), (40, 1088, 33, "32/4/3"), (40, 704, 33, "32/4/4"),
    (40, 256, 33, "32/4/4"), (4487, 128, 130, "32/8/3"), (721, 1344, 5579, "32/8/3"), (4180, 256, 147, "32/8/4"),
    (4431, 704, 137, "32/8/4"), (4250, 320, 138, "32/8/5"), (4281, 896, 129, "32/8/5"), (4394, 512, 130, "32/8/8"),
    (4354, 448, 132, "32/8/8"), (2199, 384, 3693, "64/4/3"), (8457, 896, 33, "64/4/3"), (8231, 256, 40, "64/4/4"),
    (8215, 448, 40, "64/4/4"), (8378, 128, 135, "64/8/2"), (9266, 64, 134, "64/8/2"), (15290, 1344, 146, "64/8/3"),
    (8432, 320, 134, "64/8/3"), (8663, 256, 130, "64/8/4"), (9179, 128, 262, "128/4/2"), (8649, 320, 266, "128/4/3"),
    (8710, 256, 288, "128/4/4"), (8984, 448, 261, "128/4/4"), (8508, 1344, 269, "128/4/3"), (10667, 128, 514, "128/8/2"),
    (12430, 64, 385, "128/8/2"), (7413, 576, 703, "128/8/3"), (11722, 320, 265, "128/8/3")])
def test_linear_sums_are_exact(m, k, n, cut):
    import paper_2512_05746_amd as hq

    name = "tile" if cut == "tile" else "linear (%s tokens, %s waves, units of %s)" % tuple(cut.split("/"))
    assert hq.hq_int_conv2d_kernel_name(1, 1, m, k, n, ksize=1) == name
    g = torch.Generator(device="cuda")
    g.manual_seed(m + k + n)
    xq = torch.randint(0, 256, (m, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    wq = torch.randint(0, 256, (n, 3, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    xq[m // 2] = 0x88
    wq[n // 2] = 0x88
    wq[0] = 0x77
    sx = torch.rand((m,), generator=g, device="cuda") + 0.1
    sw = torch.rand((n,), generator=g, device="cuda") * 1e-4 + 1e-5   # (three planes of 6784 channels stay finite in fp16)
    bias = torch.randn((n,), generator=g, device="cuda")

    def codes(q):
        v = torch.stack([q & 15, q >> 4], -1).flatten(-2).double()
        return torch.where(v > 7, v - 16, v)

    sums = [codes(xq) @ codes(wq[:, p]).T.contiguous() for p in range(3)]
    w0 = wq[:, 0].contiguous()
    assert torch.equal(hq.hq_int_linear(xq, sx, w0, sw, None, y_dtype=torch.int32).double(), sums[0])
    scale = sx.double()[:, None] * sw.double()
    eps = 2.0 ** -24

    def check(y, exact, size, roundings):
        limit = roundings * eps * (size + bias.double().abs())
        if y.dtype == torch.float16:
            limit = limit + exact.abs() * 2.0 ** -11 + 2.0 ** -25
        assert ((y.double() - exact).abs() <= limit).all()

    for dtype in (torch.float32, torch.float16):
        b = bias.to(dtype)
        exact = sums[0] * scale
        check(hq.hq_int_linear(xq, sx, w0, sw, b, y_dtype=dtype), exact + b.double(), exact.abs(), 4)
        exact = sums[0] * sw.double() * sx[0].double()
        check(hq.hq_int_linear_static(xq, sx[:1], w0, sw, b, y_dtype=dtype), exact + b.double(), exact.abs(), 4)
        for block, planes in ((8, 2), (64, 3)):
            norm = 1.0 / block ** 0.5
            parts = [sums[p] * scale * norm * 16.0 ** p for p in range(planes)]
            check(hq.hq_int_linear_single(xq, sx, wq, sw, b, block, y_dtype=dtype), sum(parts) + b.double(),
                  sum(q.abs() for q in parts), 8)
    y = hq.hq_int_conv2d(xq.view(1, 1, m, k // 2), sx.view(1, 1, m), w0.view(n, 1, k // 2), sw, None, ksize=1, y_dtype=torch.int32)
    assert torch.equal(y.view(m, n).double(), sums[0])


# Weights of more than 2 GiB whose steps are padded: what a padding step multiplies, and adds to the code sums, is zero wherever the
# channel lies (before, between and behind the places that 2^31 bytes from the start or from the end would reach).
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n,planes", [(40, 2368, 2000000, 1), (64, 2240, 1917500, 1), (64, 960, 1491400, 3)])
def test_linear_weights_beyond_2gib(m, k, n, planes):
    import paper_2512_05746_amd as hq

    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    wq = torch.randint(0, 256, (n, planes, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    assert wq.numel() > 1 << 31
    xq = torch.randint(0, 256, (m, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    edge = (1 << 31) // (planes * k // 2)
    at = torch.cat([torch.arange(200), edge + torch.arange(-100, 100), n - edge + torch.arange(-100, 100),
                    torch.randint(0, n, (500,)), torch.arange(n - 200, n)]).clamp(0, n - 1).cuda()

    def codes(q):
        v = torch.stack([q & 15, q >> 4], -1).flatten(-2).double()
        return torch.where(v > 7, v - 16, v)

    sums = [codes(xq) @ codes(wq[at, p]).T.contiguous() for p in range(planes)]
    if planes == 1:
        y = hq.hq_int_linear(xq, None, wq[:, 0], None, None, y_dtype=torch.int32)
        assert torch.equal(y[:, at].double(), sums[0])
        return
    sx = torch.rand((m,), generator=g, device="cuda") + 0.1
    sw = torch.rand((n,), generator=g, device="cuda") + 0.1
    y = hq.hq_int_linear_single(xq, sx, wq, sw, None, 64, y_dtype=torch.float32)
    scale = sx.double()[:, None] * sw[at].double() / 8.0
    parts = [s * scale * 16.0 ** p for p, s in enumerate(sums)]
    assert ((y[:, at].double() - sum(parts)).abs() <= 8 * 2.0 ** -24 * sum(q.abs() for q in parts)).all()


@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n,block", [(40, 128, 40, 8), (130, 640, 96, 64), (4096, 576, 1728, 64)])
def test_linear_single_of_large_token_scales(m, k, n, block):
    """Scales of up to the largest float, upper planes that are zero or not: a result is finite where the exact one is (the scale times
    the sum of a token stays below 3.4e38; two roundings of the planes' sum, three of the scales)."""
    import paper_2512_05746_amd as hq

    g = torch.Generator(device="cuda")
    g.manual_seed(m + k + n)
    xq = torch.zeros((m, k // 2), dtype=torch.uint8, device="cuda")
    xq[:, k // 4] = 1                                    # one code of 1 a token, so the sums are one weight's digits
    wq = torch.randint(0, 256, (n, 3, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    wq[: n // 2, 1:] = 0
    d = wq[:, :, k // 4].double() % 16
    total = (torch.where(d > 7, d - 16, d) * torch.tensor([1.0, 16.0, 256.0 if block > 8 else 0.0], device="cuda").double()).sum(1)
    total = total.expand(m, n)
    sw = (torch.rand((n,), generator=g, device="cuda") + 0.5) * 1e-34
    for scale in (1.2e36, 1.4e36, 4e37):
        sx = torch.full((m,), scale, device="cuda")
        y = hq.hq_int_linear_single(xq, sx, wq, sw, None, block, y_dtype=torch.float32).double()
        exact = total * sx.double()[:, None] * sw.double() / block ** 0.5
        fits = (total * scale).abs() < 3.4e38
        assert fits[:, : n // 2].all()
        assert ((y - exact).abs() <= 8 * 2.0 ** -24 * exact.abs())[fits].all()


@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [
    (1, 8, 1), (27, 40, 24),          # the kernel for few channels
    (1, 72, 1), (70, 120, 33),        # one packed dword in the last step, seven; loads that reach beyond the tensor
    (3000, 56, 440), (2100, 200, 96), (500, 952, 264), (9000, 328, 640),
    (3000, 56, 441), (2000, 104, 627),   # (int32 sums: the kernel for few channels)
    (20000, 40, 6), (16384, 40, 6),      # one group of channels out: that kernel, and not
    (2081, 4088, 1920),               # many rounds of tiles of 32 tokens
    (40, 6136, 33), (40, 6152, 33),   # the longest K of which 32 tokens fit the LDS; the kernel for few channels again
    (40, 6392, 33), (40, 8200, 33)])
def test_linear_k_no_multiple_of_64(m, k, n):
    """As above.  The codes that follow a row in memory are extreme, so that what a load finds there would show."""
    import paper_2512_05746_amd as hq

    kernel = hq.hq_int_conv2d_kernel_name(1, 1, m, k, n, ksize=1)
    assert kernel == "small-channel-count" if k > 6136 or (m, k) in ((1, 8), (27, 40), (20000, 40)) else kernel.startswith("linear (")
    g = torch.Generator(device="cuda")
    g.manual_seed(m + k + n)
    xq = torch.randint(0, 256, (m, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    wq = torch.randint(0, 256, (n, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    xq[:, :4], wq[:, :4] = 0x88, 0x88
    sx = torch.rand((m,), generator=g, device="cuda") + 0.1
    sw = torch.rand((n,), generator=g, device="cuda") * 1e-4 + 1e-5
    bias = torch.randn((n,), generator=g, device="cuda")

    def codes(q):
        v = torch.stack([q & 15, q >> 4], -1).flatten(-2).double()
        return torch.where(v > 7, v - 16, v)

    acc = codes(xq) @ codes(wq).T.contiguous()
    assert torch.equal(hq.hq_int_linear(xq, sx, wq, sw, None, y_dtype=torch.int32).double(), acc)
    for scale, call in ((sx, hq.hq_int_linear), (sx[:1], hq.hq_int_linear_static)):
        exact = acc * scale.double()[:, None] * sw.double()
        for dtype in (torch.float32, torch.float16):
            limit = 4 * 2.0 ** -24 * (exact.abs() + bias.double().abs())
            want = exact + bias.to(dtype).double()
            if dtype == torch.float16:
                limit = limit + want.abs() * 2.0 ** -11 + 2.0 ** -25
            y = call(xq, scale, wq, sw, bias.to(dtype), y_dtype=dtype)
            assert ((y.double() - want).abs() <= limit).all()
