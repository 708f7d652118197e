"""Parity of linear layers at the edges of the rule that takes 128 x 128 tiles where 64 x 128 ones need a second round: K (times
digit planes) of at least 576, more than 768 tiles of 64 x 128 and at most 512 of 128 x 128 (256 CUs).  Layers of shorter K that would
meet the rule run on the linear kernel; theirs stay here as a test of that one, and those of 1536 channels test the rule."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from parity_util import check_y, pack_codes

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("m,n,k", [
    (4096, 1536, 576),   # 768 small tiles: one round of them
    (4096, 1600, 576),   # 800: a second round, so large tiles
    (4033, 1600, 576),   # the same with a ragged last pixel tile
    (4096, 1600, 384),   # a K below the rule's
    (4096, 2048, 576),   # 512 large tiles: one round of them
    (4096, 2112, 576),   # 544: small tiles again
    (4096, 1537, 576),   # channels that are no multiple of 64 take large tiles anyway
    (4096, 1536, 1536), (4096, 1600, 1536), (4033, 1600, 1536), (4096, 2048, 1536), (4096, 2112, 1536),   # the same on the tile kernel
])
def test_linear_one_round(m, n, k):
    """Integer sums bit for bit, fp32 results to 1e-5, fp16 to 1e-3 (one rounding, 4.9e-4)."""
    import paper_2512_05746_amd as hq
    assert (hq.hq_int_conv2d_kernel_name(1, 1, m, k, n, ksize=1) == "tile") == (k == 1536)
    rng = np.random.default_rng(m + n + k)
    xq = rng.integers(-8, 8, (m, k)).astype(np.int8)
    wq = rng.integers(-8, 8, (n, k)).astype(np.int8)
    sx = rng.uniform(0.01, 0.1, m).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, n).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float16)
    acc_o, y_o = oracle.int_linear(xq, sx, wq, sw, bias)
    args = dev(pack_codes(xq)), dev(sx), dev(pack_codes(wq)), dev(sw)
    assert np.array_equal(hq.hq_int_linear(*args, None, y_dtype=torch.int32).cpu().numpy(), acc_o)
    y = hq.hq_int_linear(*args, dev(bias), y_dtype=torch.float16)
    check_y("fp16", y.cpu().numpy(), y_o, rtol=1e-3)
    y = hq.hq_int_linear(*args, dev(bias.astype(np.float32)), y_dtype=torch.float32)
    check_y("fp32", y.cpu().numpy(), y_o, rtol=1e-5)


@pytest.mark.parametrize("m,n,k,block", [
    (4096, 1600, 192, 64),   # three planes: 3 x 192 is the rule's K
    (4096, 1536, 192, 64),   # one round of small tiles
    (4033, 1600, 384, 8),    # two planes (2 x 384), ragged last pixel tile
    (4096, 1600, 192, 8),    # two planes: 2 x 192 is below the rule's K
])
def test_linear_single_one_round(m, n, k, block):
    """The Single scheme: the three integer sums bit for bit, fp32 results to 1e-5 (three folds and two roundings, each 6e-8 of
    sums of digits that may be some times the result)."""
    import paper_2512_05746_amd as hq
    rng = np.random.default_rng(m + n + k + block)
    xq = rng.integers(-8, 8, (m, k)).astype(np.int8)
    b = rng.integers(-8 * block, 8 * block + 1, (n, k))
    d0 = (b + 8) % 16 - 8
    r1 = (b - d0) // 16
    d1 = (r1 + 8) % 16 - 8
    planes = np.stack([d0, d1, (r1 - d1) // 16], axis=1)   # [n, 3, k]
    sx = rng.uniform(0.01, 0.1, m).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, n).astype(np.float32)
    args = dev(pack_codes(xq)), dev(sx), dev(pack_codes(planes.astype(np.int8))), dev(sw)
    acc = hq.hq_int_linear_single(*args, None, block, y_dtype=torch.int32).cpu().numpy()
    # (fp64 products of such sums are exact)
    want = np.stack([(xq.astype(np.float64) @ planes[:, p].T.astype(np.float64)) for p in range(3)], axis=1)
    assert np.array_equal(acc, want)
    y = hq.hq_int_linear_single(*args, None, block, y_dtype=torch.float32).cpu().numpy()
    y_o = (want[:, 0] + 16 * want[:, 1] + 256 * want[:, 2]) * sx[:, None].astype(np.float64) * sw.astype(np.float64) / block ** 0.5
    check_y("fp32", y, y_o, rtol=1e-5)
