"""The digit-plane contraction (m > 16, layouts with Had) under every plan it can take: tile shape (32 x
256, 64 x 512), parts of K, binary and ternary codes, ragged rows and columns, groups, accumulation.
Small sizes take 32 x 256 by themselves, so the small cases ask for their plan with SDQ_DIGIT_PLAN;
PLANS holds sizes that take the shapes and splits by themselves, and a test without a GPU checks that."""
import ctypes

import numpy as np
import pytest

import paper_2510_03275_amd as P
import synth
from oracle import layout as LY
from oracle import linear as OL
from tests.gpu_common import TOL, require_gpu, to_device_x

# x_tilde to 15 bits per 32 samples and random codes: 9.2e-5 of |s x_tilde|, which is |y|'s scale
# (tests/test_gpu_prefill_digits.py derives it)
BOUND = 1.4e-4

# (rows of each linear, k, OSR, m) -> (shape, splits) on 256 CUs
PLANS = [(([300], 1280, 2.0, 65), (0, 10)), (([203], 4096, 1.5, 150), (0, 16)), (([9000], 256, 1.5, 60), (0, 1)),
         (([1300, 4000, 70], 768, 1.5, 300), (0, 1)), (([10798], 256, 1.0, 1129), (1, 1)),
         (([11853, 2636, 2480], 256, 1.0, 713), (1, 1)), (([1856], 2816, 2.75, 1026), (1, 7))]


class _Plan(ctypes.Structure):
    _fields_ = [("shape", ctypes.c_int), ("splits", ctypes.c_int), ("steps_per", ctypes.c_int),
                ("part_bytes", ctypes.c_size_t)]


def _plan(ns, k_up, m, part_bytes=(1 << 64) - 1):
    """sdq::digit_plan (an internal function of the library)."""
    fn = P.lib()["_ZN3sdq10digit_planEPKlillm"]
    fn.restype = _Plan
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_size_t]
    arr = (ctypes.c_int64 * len(ns))(*ns)
    return fn(arr, len(ns), k_up, m, part_bytes)


@pytest.mark.parametrize("case,want", PLANS)
def test_plans_of_the_listed_sizes(case, want):
    ns, k, osr, m = case
    p = _plan(ns, int(k * osr), m)
    assert (p.shape, p.splits) == want


def test_plans_hold_every_part_of_k():
    rng = np.random.default_rng(5)
    for _ in range(300):
        ns = [int(n) for n in rng.integers(1, 20000, rng.integers(1, 5))]
        k_up, m = 32 * int(rng.integers(2, 1500)), int(rng.integers(17, 3000))
        steps = 2 * -(-k_up // 128)
        room = int(rng.choice([0, 1 << 20, 1 << 26, 1 << 40]))
        p = _plan(ns, k_up, m, room)
        assert p.shape in (0, 1) and p.splits >= 1 and p.steps_per % 2 == 0
        assert (p.splits - 1) * p.steps_per < steps <= p.splits * p.steps_per
        assert p.part_bytes <= room
        assert p.part_bytes == (0 if p.splits == 1 else
                                p.splits * sum(4 * (-(-m * n // 4) * 4) for n in ns))


def _encoded(torch, n, k, osr, levels, seed):
    L = P.sdq_layout_init(n, k, osr, levels)
    rng = np.random.default_rng(seed)
    codes = rng.integers(-1, 2, size=(n, L.k_up), dtype=np.int8) if levels == 3 else \
        (2 * rng.integers(0, 2, size=(n, L.k_up), dtype=np.int8) - 1)
    scales = rng.uniform(0.01, 0.02, n).astype(np.float32)
    return P.Encoded(L, torch.from_numpy(LY.pack(codes, levels)).cuda(), torch.from_numpy(scales).cuda()), codes, scales


def _check(y, x64, codes, scales, m_up):
    ref = OL.linear_fp64(x64, codes, scales, 256, m_up)
    y = y.cpu().numpy().astype(np.float64)
    assert np.all(OL.rel_err_rows(y, ref) <= TOL)
    assert np.linalg.norm(y - ref) <= BOUND * np.linalg.norm(ref)


# 17 pairs of K steps (2080 samples): parts of 34, 18 + 16, 12 + 12 + 10, 8 x 4 + 2 and 4 x 8 + 2 steps
# against a ring of four, so whole rounds and two steps over, and parts shorter than the ring.  700, 70
# and 513 columns end inside a tile and inside a panel; the m end inside and between groups of 32 rows,
# with a group missing from the last tile of two.
@pytest.mark.gpu
@pytest.mark.parametrize("levels", [2, 3])
@pytest.mark.parametrize("m", [33, 64, 70, 129])
def test_every_plan_on_ragged_groups(monkeypatch, m, levels):
    torch = require_gpu()
    ns, k, osr = [700, 70, 513], 1280, 1.625
    made = [_encoded(torch, n, k, osr, levels, n + m) for n in ns]
    L = made[0][0].layout
    x, x64 = to_device_x(synth.activations_f32(m, 6, m, k), "f16", torch)
    for splits in (1, 2, 3, 5, 9):
        seen = []
        for shape in (0, 1):
            monkeypatch.setenv("SDQ_DIGIT_PLAN", f"{shape},{splits}")
            p = _plan(ns, L.k_up, m)
            assert (p.shape, p.splits) == (shape, splits)
            ys = [torch.full((m * n + 1,), float("nan"), device="cuda")[1 - j % 2:][:m * n].view(m, n)
                  for j, n in enumerate(ns)]                 # (the first is not 16-byte aligned)
            group = P.LinearGroup([e for e, _, _ in made], ys)
            ws = torch.full((P.sdq_linear_group_workspace_bytes([e.layout for e, _, _ in made], m),), 0x7F,
                            dtype=torch.uint8, device="cuda")
            P.sdq_linear_group(x, group, ws)
            for y, (e, c, s) in zip(ys, made):
                _check(y, x64, c, s, L.m_up)
            once = [y.clone() for y in ys]
            P.sdq_linear_group(x, group, ws, accumulate=True)
            for y, o in zip(ys, once):
                assert torch.all(torch.abs(y - 2 * o) <= 2.0 ** -23 * torch.abs(2 * o))   # (scale and add may fuse)
            # the contraction alone, from the expansion that the call left
            P.sdq_linear_group_expanded(m, group, ws)
            for y, o in zip(ys, once):
                assert torch.equal(y, o)
            seen.append(once)
        for a, b in zip(*seen):
            assert torch.equal(a, b)                         # the shapes add in the same order


@pytest.mark.gpu
@pytest.mark.parametrize("levels", [2, 3])
@pytest.mark.parametrize("case,want", [c for c in PLANS if c[1][0] == 1 or c[1][1] > 1])
def test_sizes_that_take_each_plan(case, want, levels):
    torch = require_gpu()
    ns, k, osr, m = case
    made = [_encoded(torch, n, k, osr, levels, n) for n in ns]
    ys = [torch.full((m, n), float("nan"), device="cuda") for n in ns]
    group = P.LinearGroup([e for e, _, _ in made], ys)
    ws = torch.empty(P.sdq_linear_group_workspace_bytes([e.layout for e, _, _ in made], m), dtype=torch.uint8,
                     device="cuda")
    x, x64 = to_device_x(synth.activations_f32(m, 6, m, k), "bf16", torch)
    P.sdq_linear_group(x, group, ws)
    for y, (e, c, s) in zip(ys, made):
        _check(y, x64, c, s, e.layout.m_up)
