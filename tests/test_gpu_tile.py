"""Parity of linear layers at the edges of the rule that takes 128 x 128 tiles where 64 x 128 ones need a second round."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from parity_util import check_y, pack_codes

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("m,n,k", [(4000, 1537, 576), (4096, 1600, 576), (4096, 1537, 512), (4097, 1985, 576)])
def test_linear_one_round(m, n, k):
    """One tile more than a round of the small tiles, a ragged last pixel and channel tile, a K just below the rule's, one
    tile more than a round of the large ones.  fp32 results to 1e-5, fp16 to 1e-3 (one rounding, 4.9e-4)."""
    import paper_2512_05746_amd as hq
    rng = np.random.default_rng(m + n + k)
    xq = rng.integers(-8, 8, (m, k)).astype(np.int8)
    wq = rng.integers(-8, 8, (n, k)).astype(np.int8)
    sx = rng.uniform(0.01, 0.1, m).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, n).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float16)
    _, y_o = oracle.int_linear(xq, sx, wq, sw, bias)
    args = dev(pack_codes(xq)), dev(sx), dev(pack_codes(wq)), dev(sw)
    y = hq.hq_int_linear(*args, dev(bias), y_dtype=torch.float16)
    check_y("fp16", y.cpu().numpy(), y_o, rtol=1e-3)
    y = hq.hq_int_linear(*args, dev(bias.astype(np.float32)), y_dtype=torch.float32)
    check_y("fp32", y.cpu().numpy(), y_o, rtol=1e-5)
