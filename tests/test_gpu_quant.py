"""Parity of the transform-quantise kernels on the matrix cores where their cuts can go wrong."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from parity_util import check_codes, unpack_codes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k", [
    (1, 64), (17, 128), (33, 1024), (40, 960),   # few tokens: a wave for every block of the row
    (512, 256), (513, 256), (1920, 960), (1921, 960),   # about the line below which bytes stay with the butterfly
    (10912, 384), (10945, 384),                  # around 16 waves a CU of 256: one block a wave, two
    (7265, 576), (7300, 576),                    # one, three
    (12001, 832), (31993, 1024), (31993, 960),   # several groups a workgroup: one, two, three blocks a wave
    (19993, 1024), (19993, 960),                 # (too uneven for that: one group)
    (32753, 64), (32770, 320),                   # around 8 groups of 16 tokens a CU: a wave for whole tokens, its last one ragged
])
@pytest.mark.parametrize("bits,one_per_byte", [(8, True), (3, True), (4, False)])
def test_hadamard64_quant(m, k, bits, one_per_byte):
    """Codes equal the oracle's but on ties; scales to 1e-6 (sums of 64 terms in fp32, in another order); a row of zeros has scale 1."""
    import paper_2512_05746_amd as hq
    rng = np.random.default_rng(m + k + bits)
    x = rng.standard_normal((m, k)).astype(np.float16)
    x[0], x[m // 2, :] = 0, x[m // 2, :] * 50
    x_d = torch.from_numpy(x).cuda()
    xq, sx = (hq.hq_act_hadamard_quant_i8 if one_per_byte and bits != 8 else hq.hq_act_hadamard_quant)(x_d, 64, bits)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(min(m, 200)), np.arange(max(0, m - 200), m), np.arange(m // 2, min(m, m // 2 + 200))]))   # (the oracle multiplies densely)
    codes = xq.cpu().numpy()[rows]
    codes_o, s_o, t = oracle.act_hadamard_quant(x[rows], 64, bits)
    check_codes("codes", codes if one_per_byte else unpack_codes(codes), codes_o, t, bits)
    np.testing.assert_allclose(sx.cpu().numpy()[rows], s_o, rtol=1e-6)
