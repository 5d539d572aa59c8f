"""The upsampling tile of the encoder follows the launch size (64 x 32 below 1024 tiles of 128 x 64),
and the fp64 GEMM of the calibration covers symmetric products tile by tile of the lower triangle:
both sides of the rule, ragged rows and remainders."""
import numpy as np
import pytest

import oracle
import synth
from oracle import layout as LY
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


# tiles of 128 x 64: 1032, 1080 (large) and 344, 4, 2 (small); blocks of 128 and 64 on both; n past a
# tile's end
@pytest.mark.parametrize("n,k,osr,levels,block", [(300, 11008, 3.0, 3, 256), (100, 11008, 3.0, 2, 256),
                                                  (65, 512, 1.5, 3, 256), (129, 256, 2.5, 2, 128),
                                                  (190, 192, 3.5, 3, 64),
                                                  (300, 11520, 2.25, 2, 128), (300, 11520, 2.25, 3, 128),
                                                  (300, 11520, 2.5, 2, 64), (300, 11520, 2.5, 3, 64)])
def test_codes_are_exact_on_both_tiles(n, k, osr, levels, block):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    w = synth.weight_rows(n + k, 3, n, k, 0.02, True)
    r = oracle.encode(w, osr, levels, block)
    enc = P.quantize(torch.from_numpy(w).cuda(), osr, levels, block)
    assert np.array_equal(enc.scales.cpu().numpy().view(np.uint32), r.scales.view(np.uint32))
    assert np.array_equal(enc.codes.cpu().numpy(), LY.pack(r.codes, levels))


# 1, 3, 10, 45 and 153 tiles on or below the diagonal; rows that end inside a 16-deep slice
@pytest.mark.parametrize("k,m", [(64, 1), (128, 15), (256, 33), (576, 100), (1088, 257)])
def test_hessian_of_any_tile_count(k, m):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    x = torch.randn(m, k, device="cuda")
    h0 = torch.randn(k, k, dtype=torch.float64, device="cuda")
    h = h0.clone()
    P.sdq_hessian_accumulate(x, h)
    xd = x.cpu().double().numpy()
    want = h0.cpu().numpy() + 2 * (xd.T @ xd)
    # sums of m products of 24-bit numbers in fp64: (m + 2) 2^-53 of the sum of magnitudes
    bound = (m + 2) * 2.0 ** -52 * (2 * (np.abs(xd).T @ np.abs(xd)) + np.abs(h0.cpu().numpy()))
    assert np.all(np.abs(h.cpu().numpy() - want) <= bound)
