"""Prefill on FP6 digit planes (m > 16, layouts with Had): tile edges, K tails, every
input type, block size and call form, against the fp64 oracle.

The bound.  A block of 32 samples with largest magnitude in [2, 4) 2^E is kept to
2^-13 2^E, rms 2^-13 / sqrt(3) 2^E = 7.0e-5 2^E; its rms over Gaussian samples is at least
2 / 2.6 2^E, so x_tilde has a relative error of at most 9.2e-5 in the 2-norm (6e-5 on
average over the place of the maximum), and bf16 inputs add E's 2^-17.  The codes are
uncorrelated with it, so y's error relative to |y|_2 is that times the ratio of |s x_tilde|
to |y| (up to 1.5 for Sigma-Delta codes at these OSRs, whose high band adds to the former).
One fp16 rounding of x_tilde gives 2.1e-4 or more before that factor."""
import numpy as np
import pytest

import oracle
import synth
from oracle import layout as LY
from oracle import linear as OL
from tests.gpu_common import TOL, require_gpu, to_device_x

pytestmark = pytest.mark.gpu

BOUND = 1.4e-4


def _encoded(torch, n, k, osr, levels, seed, block=256, packing=0):
    import paper_2510_03275_amd as P
    r = oracle.encode(synth.weight_rows(seed, 2, n, k, 0.02, True), osr, levels, block)
    L = P.sdq_layout_init(n, k, osr, levels, block)
    buf = LY.pack(r.codes, levels)
    if packing:
        P.sdq_layout_set_packing(L, packing)
        buf = LY.pack_base3(r.codes)
    return P.Encoded(L, torch.from_numpy(buf).cuda(), torch.from_numpy(r.scales).cuda()), r


def _rel(y, y_ref):
    return np.linalg.norm(y - y_ref) / np.linalg.norm(y_ref)


def _check(y, x64, r, block=256, bound=BOUND):
    y_ref = OL.linear_fp64(x64, r.codes, r.scales, block, r.m_up)
    y = y.cpu().numpy().astype(np.float64)
    assert np.all(OL.rel_err_rows(y, y_ref) <= TOL)
    assert _rel(y, y_ref) <= bound, _rel(y, y_ref)


# whole and partial groups of 32 rows (all on 32 x 256 tiles, K split; tests/test_gpu_prefill_plans.py
# takes the other plans)
@pytest.mark.parametrize("m", [17, 32, 33, 64, 65, 96, 97, 128, 161, 192, 193, 256, 257])
@pytest.mark.parametrize("n,k,osr,levels", [(300, 1280, 2.0, 3), (257, 1280, 1.625, 2), (64, 512, 2.125, 3)])
def test_tile_edges(n, k, osr, levels, m):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    enc, r = _encoded(torch, n, k, osr, levels, seed=n + m)
    x, x64 = to_device_x(synth.activations_f32(m, 3, m, k), "f16", torch)
    _check(P.linear(x, enc), x64, r)


# K tails: k_up from one 32-sample block past a step quad to a whole number of quads
@pytest.mark.parametrize("levels", [2, 3])
@pytest.mark.parametrize("k,osr,block", [(256, 1.0, 256), (256, 1.125, 256), (768, 1.375, 256), (128, 1.25, 128),
                                         (384, 1.75, 128), (64, 1.5, 64), (320, 2.5, 64)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_k_tails_blocks_and_types(dtype, k, osr, block, levels):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    n, m = 70, 45
    enc, r = _encoded(torch, n, k, osr, levels, seed=k + levels, block=block)
    x, x64 = to_device_x(synth.activations_f32(k, 4, m, k), dtype, torch)
    _check(P.linear(x, enc), x64, r, block, bound=2 * BOUND if levels == 2 and osr < 1.5 else BOUND)


@pytest.mark.parametrize("levels,packing", [(2, 0), (3, 0), (3, 1)])
@pytest.mark.parametrize("m", [20, 150])
def test_call_forms_and_workspaces(m, levels, packing):
    """Split and unsplit contractions (full and least workspace), fp16 x_tilde where the planes do
    not fit, separate expansion and contraction, accumulation, an output that is not 16-byte aligned."""
    torch = require_gpu()
    import paper_2510_03275_amd as P
    n, k = 203, 4096
    enc, r = _encoded(torch, n, k, 1.5, levels, seed=m + levels, packing=packing)
    x, x64 = to_device_x(synth.activations_f32(m, 5, m, k), "f16", torch)
    full = P.sdq_linear_workspace_bytes(enc.layout, m)
    ws = torch.full((full,), 0x7F, dtype=torch.uint8, device="cuda")
    y = torch.full((m, n), float("nan"), device="cuda")
    P.sdq_linear(x, enc.codes, enc.scales, enc.layout, y, ws)
    _check(y, x64, r)
    again = torch.empty_like(y)
    P.sdq_linear(x, enc.codes, enc.scales, enc.layout, again, ws)
    assert torch.equal(y, again)                               # fixed order of the partial sums
    base = torch.randn(m, n, device="cuda")
    acc = base.clone()
    P.sdq_linear(x, enc.codes, enc.scales, enc.layout, acc, ws, accumulate=True)
    assert torch.max(torch.abs(acc - base - y)).item() <= 1e-5 * torch.max(torch.abs(acc)).item()
    odd = torch.empty(m * n + 1, device="cuda")[1:].view(m, n)
    P.sdq_linear(x, enc.codes, enc.scales, enc.layout, odd, ws)
    assert torch.equal(odd, y)
    # fp16 x_tilde: m x k_up, the row factors, and the unpacked codes of base-3 layouts
    chunks = -(-enc.layout.k_up // (64 if levels == 3 else 128))
    least = -(-(m * chunks * (128 if levels == 3 else 256)) // 256) * 256 + -(-(8 * m) // 256) * 256
    if packing:
        least += 256 * chunks * 16
    assert least < full
    for size, bound in ((least, 10 * BOUND), (full - 256, BOUND)):
        P.sdq_linear(x, enc.codes, enc.scales, enc.layout, odd, ws[:size])
        _check(odd, x64, r, bound=bound)
    for size in (full, least):
        P.sdq_expand_activations(x, enc.layout, ws[:size])
        P.sdq_linear_expanded(m, enc.codes, enc.scales, enc.layout, odd, ws[:size])
        _check(odd, x64, r, bound=BOUND if size == full and not packing else 10 * BOUND)
    with pytest.raises(P.SdqError) as e:
        P.sdq_linear(x, enc.codes, enc.scales, enc.layout, y, ws[:least - 1])
    assert e.value.status == -6


def test_nonfinite_activations_stay_in_their_rows():
    torch = require_gpu()
    import paper_2510_03275_amd as P
    n, k, m = 130, 768, 40
    enc, _ = _encoded(torch, n, k, 2.0, 3, seed=9)
    x = torch.randn(m, k, device="cuda").half()
    want = P.linear(x, enc)
    bad = x.clone()
    bad[3, 300], bad[17, 5], bad[39, 767] = float("inf"), float("nan"), -float("inf")
    for xb in (bad, bad.bfloat16(), bad.float()):
        y = P.linear(xb, enc)
        rows = torch.tensor([i in (3, 17, 39) for i in range(m)], device="cuda")
        assert not torch.isfinite(y[rows]).any()
        assert torch.isfinite(y[~rows]).all()
    assert torch.equal(P.linear(bad, enc)[~rows], want[~rows])


# Rows whose largest value is near the ends of fp32's normal range: below 2^-127 a block's samples are kept
# to 2^-139 only, rms 2^-141 against 2^-128 or so of the samples (1.2e-4 more than usual, twice that of the
# row's largest output); at 2^124 the sums of code times x_tilde, 16384 long and more, pass 2^128 before
# the row scale brings them back.
@pytest.mark.parametrize("levels", [2, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("e", [-126, 124])
def test_rows_at_the_ends_of_the_range(e, dtype, levels):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    n, k, m, block = 70, 16384, 20, 256
    L = P.sdq_layout_init(n, k, 1.5, levels, block)
    rng = np.random.default_rng(levels)
    codes = rng.integers(-1, 2, size=(n, L.k_up), dtype=np.int8) if levels == 3 else \
        (2 * rng.integers(0, 2, size=(n, L.k_up), dtype=np.int8) - 1)
    scales = (rng.uniform(1, 2, n) * (2.0 ** -13 if e > 0 else 1.0)).astype(np.float32)
    enc = P.Encoded(L, torch.from_numpy(LY.pack(codes, levels)).cuda(), torch.from_numpy(scales).cuda())
    x = rng.standard_normal((m, k))
    x, x64 = to_device_x(np.ldexp(x / np.abs(x).max(axis=1, keepdims=True), e).astype(np.float32), dtype, torch)
    ref = OL.linear_fp64(x64, codes, scales, block, L.m_up)
    if e > 0:
        assert np.abs(ref / scales).max() > 2.0 ** 128       # (sums that fp32 does not hold)
    err = OL.rel_err_rows(P.linear(x, enc).cpu().numpy().astype(np.float64), ref)
    assert np.all(err <= TOL), err


# more rows and columns (unsplit 32 x 256 tiles), the last column tile and row tile partial, and a group
# of linears
@pytest.mark.parametrize("ns,k,m,levels", [([9000], 256, 60, 3), ([6100], 512, 700, 2), ([12300], 512, 1500, 3),
                                           ([1300, 4000, 70], 768, 300, 3), ([2100], 4096, 900, 2)])
def test_tile_shapes_and_groups(ns, k, m, levels):
    torch = require_gpu()
    import paper_2510_03275_amd as P
    made = [_encoded(torch, n, k, 1.5, levels, seed=n) for n in ns]
    ys = [torch.full((m, n), float("nan"), device="cuda") for n in ns]
    group = P.LinearGroup([e for e, _ in made], ys)
    ws = torch.empty(P.sdq_linear_group_workspace_bytes([e.layout for e, _ in made], m), dtype=torch.uint8,
                     device="cuda")
    x, x64 = to_device_x(synth.activations_f32(m, 6, m, k), "bf16", torch)
    P.sdq_linear_group(x, group, ws)
    for y, (_, r) in zip(ys, made):
        _check(y, x64, r)
