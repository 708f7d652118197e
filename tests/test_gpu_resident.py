"""Parity of the activation-resident kernel (4-bit codes, stride 1) at the sizes where its cuts can go wrong."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from parity_util import check_codes, check_y, pack_codes, unpack_codes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hq():
    import paper_2512_05746_amd as mod
    return mod


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (1, 1, 1, 64, 1),          # one pixel, one channel: a single 64-channel step, every tap but one outside
    (1, 5, 127, 128, 33),      # two steps per slice; one pixel short of a tile; one channel in the second block
    (2, 8, 8, 320, 96),        # five steps in slices of three: the last slice is padded
    (3, 43, 1, 192, 160),      # images one pixel wide; one pixel more than a tile; five blocks in three phases
    (1, 6, 200, 960, 40),      # rows so long that only some slices are resident at a time
    (2, 33, 60, 448, 72),      # two pixel groups or one, padded slice, ragged channels
    (5, 40, 40, 256, 200),     # seven channel blocks
])
def test_conv3x3(hq, nb, h, w, cin, cout):
    """Per-tap sums and the sum over all taps bit for bit (the fp32 sums of the 6-bit instruction are exact below 2^24);
    fp32 results to 1e-5 of the largest (nine folds, or eighteen where only some slices are resident at a time, and few
    roundings more, each 6e-8 of partial sums, which with codes of both signs may be some times larger than it)."""
    rng = np.random.default_rng(nb * 1000 + h * 100 + w + cin + cout)
    xq = rng.integers(-8, 8, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-8, 8, (cout, 3, 3, cin)).astype(np.int8)
    xq[0, 0, 0, :], wq[0, :, :, :] = -8, -8
    sx = rng.uniform(0.01, 1.0, (nb, h, w)).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, cout).astype(np.float32)
    bias = rng.standard_normal(cout).astype(np.float32)
    xq_d, wq_d = dev(pack_codes(xq)), dev(pack_codes(wq.reshape(cout, 9, cin)))
    acc_o, y_o = oracle.int_conv2d(xq, sx, wq, sw, bias, stride=1, pad=1)
    acc = host(hq.hq_int_conv2d(xq_d, None, wq_d, None, None, ksize=3, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o), "per-tap sums"
    acc = host(hq.hq_int_conv2d_static(xq_d, None, wq_d, None, None, ksize=3, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o.sum(axis=3)), "one sum"
    y = host(hq.hq_int_conv2d(xq_d, dev(sx), wq_d, dev(sw), dev(bias), ksize=3, y_dtype=torch.float32))
    check_y("y", y, y_o, rtol=1e-5)
    s1 = torch.tensor([0.37], dtype=torch.float32, device="cuda")
    _, y_o = oracle.int_conv2d_static(xq, 0.37, wq, sw, bias, stride=1, pad=1, want_acc=False)
    y = host(hq.hq_int_conv2d_static(xq_d, s1, wq_d, dev(sw), dev(bias), ksize=3, y_dtype=torch.float32))
    check_y("y (static)", y, y_o, rtol=1e-5)


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (2, 16, 16, 64, 64),         # one slice: one unit a tap
    (1, 20, 13, 128, 33),        # two steps in one slice
    (2, 9, 9, 960, 200),         # five slices, taps cut between the waves that share a task
    (4, 16, 16, 576, 576),       # three slices
    (1, 6, 200, 960, 40),        # some slices resident at a time
    (3, 45, 27, 320, 200),       # a padded slice, seven channel blocks
])
def test_conv3x3_fp32_codes_of_one_sign(hq, nb, h, w, cin, cout):
    """fp32 results with per-pixel scales where the weights' offset of 8 times the sum of the activation codes is far larger
    than the result: no digits may be lost to it.  No partial sum exceeds the result's size by more than a tap's, so the bound
    is 20 roundings of 2^-24 (nine folds, or eighteen where the tile holds only part of the slices; scale and bias)."""
    rng = np.random.default_rng(cin + cout)
    xq = rng.integers(3, 8, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-1, 3, (cout, 3, 3, cin)).astype(np.int8)
    sx = rng.uniform(0.1, 1.0, (nb, h, w)).astype(np.float32)
    sw = rng.uniform(0.05, 0.1, cout).astype(np.float32)
    _, y_o = oracle.int_conv2d(xq, sx, wq, sw, None, stride=1, pad=1, want_acc=False)
    y = host(hq.hq_int_conv2d(dev(pack_codes(xq)), dev(sx), dev(pack_codes(wq.reshape(cout, 9, cin))), dev(sw), None, ksize=3,
                              y_dtype=torch.float32))
    check_y("y", y, y_o, rtol=20 * 2.0 ** -24)


@pytest.mark.parametrize("scale", [1e37, 1e-30])
def test_conv3x3_extreme_scales(hq, scale):
    """Scales near the ends of fp32's range whose products with the weights' are ordinary numbers."""
    rng = np.random.default_rng(5)
    nb, h, w, cin, cout = 2, 9, 9, 384, 40
    xq = np.zeros((nb, h, w, cin), np.int8)
    xq[..., :3] = rng.integers(-1, 2, (nb, h, w, 3))     # (sums of up to 27 codes: no product of scale and sum overflows)
    wq = rng.integers(-1, 2, (cout, 3, 3, cin)).astype(np.int8)
    sx = (rng.uniform(0.5, 1.0, (nb, h, w)) * scale).astype(np.float32)
    sw = (rng.uniform(0.5, 1.0, cout) / scale).astype(np.float32)
    _, y_o = oracle.int_conv2d(xq, sx, wq, sw, None, stride=1, pad=1, want_acc=False)
    for ydt, rtol in ((torch.float32, 1e-5), (torch.float16, 1e-3)):
        y = hq.hq_int_conv2d(dev(pack_codes(xq)), dev(sx), dev(pack_codes(wq.reshape(cout, 9, cin))), dev(sw), None, ksize=3, y_dtype=ydt)
        check_y("y", host(y), y_o, rtol=rtol)


@pytest.mark.parametrize("nb,h,w,cin,cout,block", [
    (1, 3, 8, 64, 1, 8),         # two planes; one channel
    (2, 5, 16, 128, 40, 16),     # two steps per slice
    (1, 7, 64, 320, 96, 32),     # upper digits up to +-16, padded slice
    (2, 9, 48, 960, 72, 16),     # the largest sums that go this way; some slices resident at a time
    (1, 3, 48, 192, 33, 1),      # no transform
    (1, 2, 64, 512, 40, 32),     # sums beyond 2^24: the tile kernel
    (1, 3, 208, 192, 40, 16),    # the longest rows that fit beside 16-pixel blocks
    (1, 3, 224, 192, 40, 16),    # rows too long: the tile kernel, three planes
    (1, 3, 216, 192, 40, 8),     # and two
])
def test_conv_width(hq, nb, h, w, cin, cout, block):
    """Integer sums bit for bit, extreme numbers (+-8 x block) among them; fp32 results to 1e-6 (three roundings)."""
    rng = np.random.default_rng(nb * 1000 + h * 100 + w + cin + cout + block)
    q = rng.integers(-8, 8, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-8, 8, (cout, 3, 3, cin)).astype(np.int8)
    q[0, 0, :, : cin // 2], wq[0] = -8, 7   # a flat line: one number of -8 x block
    signs = np.ones(block)
    for b in range(block.bit_length() - 1):
        signs *= np.where(np.arange(block) >> b & 1, -1, 1)
    q[-1, -1, :, cin // 2:] = np.tile(np.where(signs < 0, -8, 7), w // block)[:, None]   # nearly +8 x block
    hb = np.array([[(-1) ** bin(i & j).count("1") for j in range(block)] for i in range(block)])
    u = np.einsum("nhbic,ij->nhbjc", q.astype(np.int64).reshape(nb, h, w // block, block, cin), hb).reshape(nb, h, w, cin)
    d0 = (u + 8) % 16 - 8
    r1 = (u - d0) // 16
    d1 = (r1 + 8) % 16 - 8
    planes = dev(pack_codes(np.stack([d0, d1, (r1 - d1) // 16]).astype(np.int8)))
    sw = rng.uniform(0.001, 0.1, cout).astype(np.float32)
    bias = rng.standard_normal(cout).astype(np.float32)
    wq_d = dev(pack_codes(wq.reshape(cout, 9, cin)))
    s1 = torch.tensor([0.37], dtype=torch.float32, device="cuda")
    acc_o, y_o = oracle.int_conv2d_width(q, 0.37, wq, sw, block, bias, stride=1, pad=1)
    acc = host(hq.hq_int_conv2d_width(planes, None, wq_d, None, None, block, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o)
    y = host(hq.hq_int_conv2d_width(planes, s1, wq_d, dev(sw), dev(bias), block, y_dtype=torch.float32))
    check_y("y", y, y_o, rtol=1e-6)


@pytest.mark.parametrize("block", [1, 8, 16, 32])
def test_conv_width_whole_range(hq, block):
    """Every integer of -8 x block .. 8 x block in the planes, wherever it comes from: integer sums bit for bit."""
    rng = np.random.default_rng(block)
    nb, h, w, cin, cout = 1, 3, 64, 128, 40
    top = 8 * block
    u = rng.integers(-top, top + 1, (nb, h, w, cin))
    u.reshape(-1)[: 2 * top + 1] = np.arange(-top, top + 1)
    d0 = (u + 8) % 16 - 8
    r1 = (u - d0) // 16
    d1 = (r1 + 8) % 16 - 8
    planes = dev(pack_codes(np.stack([d0, d1, (r1 - d1) // 16]).astype(np.int8)))
    wq = rng.integers(-8, 8, (cout, 9, cin)).astype(np.int8)
    up = np.pad(u, ((0, 0), (1, 1), (1, 1), (0, 0)))
    want = sum(up[:, t // 3:t // 3 + h, t % 3:t % 3 + w] @ wq[:, t].astype(np.int64).T for t in range(9))
    acc = host(hq.hq_int_conv2d_width(planes, None, dev(pack_codes(wq)), None, None, block, y_dtype=torch.int32))
    assert np.array_equal(acc, want)


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (1, 1, 1, 64, 1),          # one pixel, one channel: a single 64-channel step
    (1, 5, 127, 128, 33),      # two steps per slice; one pixel short of a tile; one channel in the second block
    (3, 43, 1, 320, 160),      # images one pixel wide; the last slice is padded; five blocks
    (1, 6, 200, 960, 40),      # rows so long that only some slices are resident at a time
    (2, 33, 60, 448, 72),      # padded slice, ragged channels
])
def test_conv3x3_8bit(hq, nb, h, w, cin, cout):
    """8-bit codes, extreme ones among them: per-tap sums bit for bit (within 192 channels they stay below 2^24); fp32
    results to 1e-5: at most nine folds a slice and two roundings more, each 6e-8 of sums below 8 x the result's."""
    rng = np.random.default_rng(nb * 1000 + h * 100 + w + cin + cout)
    xq = rng.integers(-128, 128, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-128, 128, (cout, 3, 3, cin)).astype(np.int8)
    xq[0, 0, 0, :], wq[0, :, :, :] = -128, -128
    sx = rng.uniform(0.01, 1.0, (nb, h, w)).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, cout).astype(np.float32)
    bias = rng.standard_normal(cout).astype(np.float32)
    xq_d, wq_d = dev(xq), dev(wq.reshape(cout, 9, cin))
    acc_o, y_o = oracle.int_conv2d(xq, sx, wq, sw, bias, stride=1, pad=1)
    acc = host(hq.hq_int_conv2d_i8(xq_d, None, wq_d, None, None, ksize=3, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o), "per-tap sums"
    y = host(hq.hq_int_conv2d_i8(xq_d, dev(sx), wq_d, dev(sw), dev(bias), ksize=3, y_dtype=torch.float32))
    check_y("y", y, y_o, rtol=1e-5)


@pytest.mark.parametrize("h,w,cin,cout,kernel", [
    (4, 1344, 64, 40, "resident"), (4, 1345, 64, 40, "tile"),     # the longest image row whose tile fits, and one more
    (4, 454, 320, 72, "resident"), (4, 455, 320, 72, "tile"),     # (slices in turn; fp32 results: tile on both sides)
    (4, 207, 960, 40, "resident"), (4, 208, 960, 40, "tile"),     # estimated to be faster on the tile kernel
    (24, 320, 576, 72, "tile"), (32, 256, 384, 208, "tile"),      # K chunks of 192 codes, ragged channels
    (90, 256, 192, 192, "tile"),                                  # 64 x 128 tiles
])
def test_conv3x3_long_rows(hq, h, w, cin, cout, kernel):
    """Both sides of the rule between the resident and the tile kernel: per-tap sums and one sum bit for bit, fp32 and fp16
    results (1e-5: eighteen folds at most and few roundings more, partial sums up to some times the result; 1e-3: fp16)."""
    rng = np.random.default_rng(h + w + cin + cout)
    name = hq.hq_int_conv2d_kernel_name(1, h, w, cin, cout)
    assert name == "tile" if kernel == "tile" else name.startswith("activation-resident"), name
    xq = rng.integers(-8, 8, (1, h, w, cin)).astype(np.int8)
    wq = rng.integers(-8, 8, (cout, 3, 3, cin)).astype(np.int8)
    sx = rng.uniform(0.01, 1.0, (1, h, w)).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, cout).astype(np.float32)
    bias = rng.standard_normal(cout).astype(np.float16)
    xq_d, wq_d = dev(pack_codes(xq)), dev(pack_codes(wq.reshape(cout, 9, cin)))
    acc_o, y_o = oracle.int_conv2d(xq, sx, wq, sw, bias, stride=1, pad=1)
    acc = host(hq.hq_int_conv2d(xq_d, None, wq_d, None, None, ksize=3, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o), "per-tap sums"
    acc = host(hq.hq_int_conv2d_static(xq_d, None, wq_d, None, None, ksize=3, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o.sum(axis=3)), "one sum"
    for ydt, rtol in ((torch.float32, 1e-5), (torch.float16, 1e-3)):
        b = dev(bias).to(ydt)
        check_y("y", host(hq.hq_int_conv2d(xq_d, dev(sx), wq_d, dev(sw), b, ksize=3, y_dtype=ydt)), y_o, rtol=rtol)
    s1 = torch.tensor([0.37], dtype=torch.float32, device="cuda")
    _, y_o = oracle.int_conv2d_static(xq, 0.37, wq, sw, bias, stride=1, pad=1, want_acc=False)
    y = host(hq.hq_int_conv2d_static(xq_d, s1, wq_d, dev(sw), dev(bias), ksize=3, y_dtype=torch.float16))
    check_y("y (static)", y, y_o, rtol=1e-3)


@pytest.mark.parametrize("h,w,cin,cout,kernel", [
    (4, 329, 192, 40, "resident"), (4, 330, 192, 40, "tile"), (4, 1031, 64, 40, "resident"), (4, 1032, 64, 40, "tile"),
    (4, 329, 960, 40, "resident"), (90, 256, 192, 192, "tile"),
])
def test_conv3x3_8bit_long_rows(hq, h, w, cin, cout, kernel):
    """As test_conv3x3_long_rows."""
    rng = np.random.default_rng(h + w + cin + cout)
    name = hq.hq_int_conv2d_kernel_name(1, h, w, cin, cout, bits=8)
    assert name == "tile" if kernel == "tile" else name.startswith("activation-resident"), name
    xq = rng.integers(-128, 128, (1, h, w, cin)).astype(np.int8)
    wq = rng.integers(-128, 128, (cout, 3, 3, cin)).astype(np.int8)
    sx = rng.uniform(0.01, 1.0, (1, h, w)).astype(np.float32)
    sw = rng.uniform(1e-5, 1e-3, cout).astype(np.float32)   # (fp16 results stay in range)
    xq_d, wq_d = dev(xq), dev(wq.reshape(cout, 9, cin))
    acc_o, y_o = oracle.int_conv2d(xq, sx, wq, sw, None, stride=1, pad=1)
    acc = host(hq.hq_int_conv2d_i8(xq_d, None, wq_d, None, None, ksize=3, y_dtype=torch.int32))
    assert np.array_equal(acc, acc_o), "per-tap sums"
    for ydt, rtol in ((torch.float32, 1e-5), (torch.float16, 1e-3)):
        check_y("y", host(hq.hq_int_conv2d_i8(xq_d, dev(sx), wq_d, dev(sw), None, ksize=3, y_dtype=ydt)), y_o, rtol=rtol)


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("w,c,block", [
    (6, 2, 2),        # one channel pair
    (8, 6, 8),        # no whole quad of pairs: bytes
    (12, 8, 4),       # one quad, one pixel group
    (64, 24, 64),     # the largest block; three quads
    (16, 1032, 16),   # more pairs than a workgroup's threads, the second pass nearly empty
    (5, 520, 1),      # no transform
])
def test_width_quant(hq, dtype, w, c, block):
    """The planes hold q H_raw exactly for codes q that are the oracle's (but for values on a rounding tie)."""
    rng = np.random.default_rng(w + c + block)
    x = rng.standard_normal((2, 3, w, c)).astype(dtype)
    scale = 0.3   # clamps at both ends
    q_o, t = oracle.act_width_quant_static(x, block, 4, float(np.float32(scale)))
    xu3 = host(hq.hq_act_hadamard_quant_width(dev(x), torch.tensor([scale], device="cuda"), block, 4))
    d = unpack_codes(xu3).astype(np.int64)
    hb = np.array([[(-1) ** bin(i & j).count("1") for j in range(block)] for i in range(block)])
    u = (d[0] + 16 * d[1] + 256 * d[2]).reshape(2, 3, w // block, block, c)
    back = np.einsum("nhbic,ij->nhbjc", u, hb).reshape(x.shape)
    assert (back % block == 0).all()
    check_codes("codes", (back // block).astype(np.int8), q_o, t, 4)


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (1, 1, 1, 64, 33),          # every tap but one outside
    (2, 3, 8, 192, 40),         # shares of a few steps, fewer than the ring holds
    (1, 46, 46, 960, 72),       # all slices resident, no room for a ring of weights
    (1, 6, 200, 960, 40),       # some slices resident at a time, nor room
    (1, 3, 32, 960, 40),        # all slices, a ring of two slots
    (1, 3, 48, 960, 40),        # some at a time, a ring of three slots
    (1, 3, 56, 960, 40),        # and of two
    (1, 5, 212, 768, 40),       # three steps at a time, unrolled
])
def test_conv3x3_one_scale_empty_sums(hq, nb, h, w, cin, cout):
    """Pixels whose window holds only zeros give exactly the bias, also where codes lie just outside the image (the rows above
    and below, the other end of the neighbouring lines): whatever a tap outside leaves in a sum has to be gone."""
    assert hq.hq_int_conv2d_kernel_name(nb, h, w, cin, cout, static_scale=True).endswith("in turn)") == (w in (200, 48, 56, 212))
    rng = np.random.default_rng(h + w + cin)
    wq = rng.integers(-8, 8, (cout, 9, cin)).astype(np.int8)
    sw = rng.uniform(0.001, 0.1, cout).astype(np.float32)
    s1 = torch.tensor([0.37], dtype=torch.float32, device="cuda")
    xq = np.zeros((nb, h, w, cin), np.int8)
    for bias in (np.zeros(cout, np.float32), rng.standard_normal(cout).astype(np.float32)):
        y = host(hq.hq_int_conv2d_static(dev(pack_codes(xq)), s1, dev(pack_codes(wq)), dev(sw), dev(bias), ksize=3, y_dtype=torch.float32))
        assert np.array_equal(y, np.broadcast_to(bias, y.shape))
    if w < 4:
        return
    xq[:, :, w // 2 + 2:] = rng.integers(-8, 8, xq[:, :, w // 2 + 2:].shape)   # (the left edge's neighbours in memory)
    acc_o, y_o = oracle.int_conv2d_static(xq, 0.37, wq.reshape(cout, 3, 3, cin), sw, None, stride=1, pad=1)
    y = host(hq.hq_int_conv2d_static(dev(pack_codes(xq)), s1, dev(pack_codes(wq)), dev(sw), None, ksize=3, y_dtype=torch.float32))
    assert (y[:, :, : w // 2] == 0).all()
    check_y("y", y, y_o, rtol=1e-5)   # (fp32: sums are exact, three roundings)


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (2, 7, 8, 64, 40), (1, 33, 24, 128, 33), (3, 9, 16, 192, 72), (2, 7, 8, 256, 40),   # taps of one to four steps: unrolled
    (2, 7, 8, 320, 40),          # five: a loop, the second item of the fill is not whole
    (7, 24, 40, 192, 200),       # two pixel groups a workgroup, several phases
    (1, 243, 136, 384, 8),       # three steps resident at a time, with per-pixel scales and on the width axis
    (1, 3, 56, 960, 40),         # one scale: a ring of two slots
    (1, 3, 88, 448, 40),         # per-pixel scales: a ring of two slots
    (1, 3, 88, 960, 40),         # and nine steps resident at a time
    (1, 3, 24, 640, 40),         # 8 bits: a ring of two slots
    (1, 13, 13, 576, 40),        # few workgroups of four waves: all of the LDS for each
    (2, 9, 16, 448, 40), (1, 16, 16, 512, 72),   # groups of three steps and one, and two, by themselves; shares that start within a tap
    (1, 3, 56, 704, 40),         # one scale: nine steps resident, then two
    (1, 5, 72, 832, 40),         # and thirteen steps in all: nine and four, or six, six and one
])
def test_conv3x3_steps_of_a_tap(hq, nb, h, w, cin, cout):
    """Every form, unrolled and not, with every type of results: integer sums bit for bit, fp32 results to 1e-5 of the largest (the width
    axis 1e-6, three roundings), fp16 to 1e-3 (one rounding, 4.9e-4)."""
    rng = np.random.default_rng(nb * 1000 + h * 100 + w + cin + cout)
    if (w, cin) in ((136, 384), (88, 960)):
        assert hq.hq_int_conv2d_kernel_name(nb, h, w, cin, cout).endswith("slices in turn)")
    sx = rng.uniform(0.01, 1.0, (nb, h, w)).astype(np.float32)
    sw = rng.uniform(1e-5, 1e-3, cout).astype(np.float32)   # (fp16 results of 8-bit codes stay in range)
    bias = rng.standard_normal(cout).astype(np.float16)
    s1 = torch.tensor([0.37], dtype=torch.float32, device="cuda")

    def check(call, x, scale, q_w, acc_o, y_o, rtol, *block):
        assert np.array_equal(host(call(x, None, q_w, None, None, *block, y_dtype=torch.int32)), acc_o)
        for ydt, tol in ((torch.float32, rtol), (torch.float16, 1e-3)):
            check_y("y", host(call(x, scale, q_w, dev(sw), dev(bias).to(ydt), *block, y_dtype=ydt)), y_o, rtol=tol)

    xq = rng.integers(-8, 8, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-8, 8, (cout, 3, 3, cin)).astype(np.int8)
    xq[0, 0, 0, :], wq[0, :, :, :] = -8, -8
    x4, w4 = dev(pack_codes(xq)), dev(pack_codes(wq.reshape(cout, 9, cin)))
    acc_o, y_o = oracle.int_conv2d(xq, sx, wq, sw, bias, stride=1, pad=1)
    check(hq.hq_int_conv2d, x4, dev(sx), w4, acc_o, y_o, 1e-5)
    acc_o, y_o = oracle.int_conv2d_static(xq, 0.37, wq, sw, bias, stride=1, pad=1)
    check(hq.hq_int_conv2d_static, x4, s1, w4, acc_o, y_o, 1e-5)
    block = 8 if w % 8 == 0 else 1
    hb = np.array([[(-1) ** bin(i & j).count("1") for j in range(block)] for i in range(block)])
    u = np.einsum("nhbic,ij->nhbjc", xq.astype(np.int64).reshape(nb, h, w // block, block, cin), hb).reshape(nb, h, w, cin)
    d0 = (u + 8) % 16 - 8
    r1 = (u - d0) // 16
    d1 = (r1 + 8) % 16 - 8
    planes = dev(pack_codes(np.stack([d0, d1, (r1 - d1) // 16]).astype(np.int8)))
    acc_o, y_o = oracle.int_conv2d_width(xq, 0.37, wq, sw, block, bias, stride=1, pad=1)
    check(hq.hq_int_conv2d_width, planes, s1, w4, acc_o, y_o, 1e-6, block)
    xq = rng.integers(-128, 128, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-128, 128, (cout, 3, 3, cin)).astype(np.int8)
    acc_o, y_o = oracle.int_conv2d(xq, sx, wq, sw, bias, stride=1, pad=1)
    check(hq.hq_int_conv2d_i8, dev(xq), dev(sx), dev(wq.reshape(cout, 9, cin)), acc_o, y_o, 1e-5)


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (1, 1, 1, 8, 1),             # one packed dword a tap; the loads of the last tap reach beyond the tensor
    (2, 9, 8, 72, 40), (1, 12, 24, 184, 33),   # two and three steps a tap, unrolled; seven packed dwords in the last
    (3, 9, 16, 248, 72),         # four, unrolled for codes
    (2, 16, 16, 328, 200),       # six steps: shares begin within a tap
    (1, 33, 24, 456, 40), (2, 8, 8, 952, 96),  # eight and fifteen
    (1, 3, 88, 952, 40),         # some resident at a time
    (1, 4, 300, 200, 40),        # the tile takes nearly all of the LDS
    (1, 2, 1500, 200, 40),       # rows too long: the kernel for few channels
])
def test_conv3x3_channels_no_multiple_of_64(hq, nb, h, w, cin, cout):
    """As test_conv3x3_steps_of_a_tap.  Weights of -8 follow the end of every row, so that what a load finds there would show."""
    for static_scale in (False, True):
        kernel = hq.hq_int_conv2d_kernel_name(nb, h, w, cin, cout, static_scale=static_scale)
        assert kernel == "small-channel-count" if w == 1500 else kernel.startswith("activation-resident (")
    rng = np.random.default_rng(nb * 1000 + h * 100 + w + cin + cout)
    xq = rng.integers(-8, 8, (nb, h, w, cin)).astype(np.int8)
    wq = rng.integers(-8, 8, (cout, 3, 3, cin)).astype(np.int8)
    wq[..., :8], xq[..., :8] = -8, 7
    sx = rng.uniform(0.01, 1.0, (nb, h, w)).astype(np.float32)
    sw = rng.uniform(1e-5, 1e-3, cout).astype(np.float32)
    bias = rng.standard_normal(cout).astype(np.float16)
    x4, w4 = dev(pack_codes(xq)), dev(pack_codes(wq.reshape(cout, 9, cin)))
    s1 = torch.tensor([0.37], dtype=torch.float32, device="cuda")
    for call, scale, (acc_o, y_o) in (
            (hq.hq_int_conv2d, dev(sx), oracle.int_conv2d(xq, sx, wq, sw, bias, stride=1, pad=1)),
            (hq.hq_int_conv2d_static, s1, oracle.int_conv2d_static(xq, 0.37, wq, sw, bias, stride=1, pad=1))):
        assert np.array_equal(host(call(x4, None, w4, None, None, ksize=3, y_dtype=torch.int32)), acc_o)
        for ydt, tol in ((torch.float32, 1e-5), (torch.float16, 1e-3)):
            check_y("y", host(call(x4, scale, w4, dev(sw), dev(bias).to(ydt), ksize=3, y_dtype=ydt)), y_o, rtol=tol)


@pytest.mark.parametrize("nb,h,w,cin,cout", [
    (1, 1, 1, 8, 2), (2, 9, 8, 72, 40), (1, 12, 24, 184, 34), (3, 9, 16, 248, 72), (2, 16, 16, 328, 200), (2, 8, 8, 952, 96),
    (1, 3, 88, 952, 40)])
def test_conv3x3_channels_no_multiple_of_64_rounded_once(hq, nb, h, w, cin, cout):
    """Per-pixel scales, fp16 and fp32 results: no further from the exact result than the sums of taps in integers, combined in fp32, are,
    that is 32 roundings (a fold or two a tap, 7 sums of waves, the scales) of at most the sum of the terms' magnitudes, and one to the
    type of the result.  Codes of one sign, and weights whose sum is zero over constant codes: the terms of half of the channels are
    zero in half of the images' rows, and so is the result, whatever offset the weights carry on the way."""
    rng = np.random.default_rng(nb * 1000 + h * 100 + w + cin + cout)
    xq = rng.integers(0, 8, (nb, h, w, cin)).astype(np.int8)
    xq[:, : (h + 1) // 2] = 7
    wq = rng.integers(-8, 8, (cout, 3, 3, cin)).astype(np.int8)
    wq[::2] = np.tile([7, -7], cin // 2)
    sx = rng.uniform(0.01, 1.0, (nb, h, w)).astype(np.float32)
    sw = rng.uniform(0.1, 1.0, cout).astype(np.float32)
    acc, _ = oracle.int_conv2d(xq, sx, wq, sw, None, stride=1, pad=1)
    padded = np.pad(sx.astype(np.float64), ((0, 0), (1, 1), (1, 1)))
    under = np.stack([padded[:, t // 3:t // 3 + h, t % 3:t % 3 + w] for t in range(9)], axis=-1)   # [nb, h, w, tap]
    terms = acc * under[..., None] * sw.astype(np.float64)
    want, limit = terms.sum(axis=3), 32 * 2.0 ** -24 * np.abs(terms).sum(axis=3)
    x4, w4 = dev(pack_codes(xq)), dev(pack_codes(wq.reshape(cout, 9, cin)))
    for dtype, half_ulp, least in ((torch.float32, 2.0 ** -24, 0.0), (torch.float16, 2.0 ** -11, 2.0 ** -25)):
        y = host(hq.hq_int_conv2d(x4, dev(sx), w4, dev(sw), None, ksize=3, y_dtype=dtype)).astype(np.float64)
        assert (np.abs(y - want) <= limit + half_ulp * np.abs(want) + least * (want != 0)).all()
