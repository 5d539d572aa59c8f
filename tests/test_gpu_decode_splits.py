"""9-16-row decodes take one block per wave on launches that fit the chip at once and two on larger
ones: both sides of the rule (1042 and 94 workgroups at one block per wave), a panel and a K split
that end early, against the fp64 definition on random codes."""
import numpy as np
import pytest

import synth
from oracle import layout as LY
from oracle import linear as OL
from tests.gpu_common import TOL, require_gpu, to_device_x

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [9, 12, 16])
@pytest.mark.parametrize("n", [33300, 3000])
def test_splits_of_both_launch_sizes(n, m):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    k, osr = 1280, 1.625
    L = P.sdq_layout_init(n, k, osr, 3)
    rng = np.random.default_rng(n + m)
    codes = rng.integers(-1, 2, size=(n, L.k_up), dtype=np.int8)
    scales = rng.uniform(0.01, 0.02, n).astype(np.float32)
    enc = P.Encoded(L, torch.from_numpy(LY.pack(codes, 3)).cuda(), torch.from_numpy(scales).cuda())
    x, x64 = to_device_x(synth.activations_f32(m, 1, m, k), "f16", torch)
    y = P.linear(x, enc).cpu().numpy().astype(np.float64)
    err = OL.rel_err_rows(y, OL.linear_fp64(x64, codes, scales, 256, L.m_up))
    assert np.all(err <= 1e-2 * TOL), err.max()       # 24-bit planes: 1e-5, as the decode path's figure


# 2-bit fields in batches of one step and of four, binary and base-3 codes, on both sides
@pytest.mark.parametrize("m", [10, 16])
@pytest.mark.parametrize("n", [33300, 28000, 3000])
@pytest.mark.parametrize("osr,levels,packing", [(2.0, 3, 0), (2.0, 2, 0), (1.625, 3, 1)])
def test_splits_of_every_storage(osr, levels, packing, n, m):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    k = 1280
    L = P.sdq_layout_init(n, k, osr, levels)
    rng = np.random.default_rng(n + m)
    codes = rng.integers(-1, 2, size=(n, L.k_up), dtype=np.int8) if levels == 3 else \
        (2 * rng.integers(0, 2, size=(n, L.k_up), dtype=np.int8) - 1)
    buf = LY.pack(codes, levels)
    if packing:
        P.sdq_layout_set_packing(L, packing)
        buf = LY.pack_base3(codes)
    scales = rng.uniform(0.01, 0.02, n).astype(np.float32)
    enc = P.Encoded(L, torch.from_numpy(buf).cuda(), torch.from_numpy(scales).cuda())
    x, x64 = to_device_x(synth.activations_f32(m, 1, m, k), "f16", torch)
    y = P.linear(x, enc).cpu().numpy().astype(np.float64)
    err = OL.rel_err_rows(y, OL.linear_fp64(x64, codes, scales, 256, L.m_up))
    assert np.all(err <= 1e-2 * TOL), err.max()
