"""Systematic errors of the float32 transforms: the mean over channels of the zero lag's error, whose exact value is the
sum of |x|^2 of the integer samples."""

import math
import sys

import pytest
import torch

import paper_0909_0001_amd as omni

pytestmark = pytest.mark.gpu

LEVELS = [[[16, 16]], [[5, 5]], [[10, 2], [5, 3]], [[12, 12]], [[9, 8], [2, 3]], [[6, 3], [3, 3]], [[4, 4], [8, 3]]]


@pytest.mark.parametrize("levels", LEVELS)
def test_zero_lags_are_unbiased(levels):
    """Rotations of exact length leave the sum of all powers alone; rounding errors have no sign and average out over
    the cells and channels.  Twiddles rounded to float32 make -3.3e-8 an axis of 12, -3.7e-8 of 9, -2.7e-8 of 8,
    -2.1e-8 of 3, +2.8e-8 of 5; the bar is below the smallest.  The powers are read from the integration state (float64): a float32
    visibility of more than 24 bits lies on a tie for every second integer, which the sign of any error decides."""
    F, T, N = 64, 16, math.prod(n for lvl in levels for n in lvl)
    gen = torch.Generator().manual_seed(N)
    raw = torch.randint(-127, 128, (T, F, N, 2), generator=gen, dtype=torch.int16).to(torch.int8)
    print("zero lags", levels, file=sys.stderr, flush=True)
    plan = omni.Plan(levels, None, F, "ci8", "fp32")
    plan.correlate(raw.cuda())
    state = torch.empty(plan.accumulator_bytes() // 8, dtype=torch.float64)
    plan.accumulator_get(state)
    got = state.reshape(F, -1).mean(1).numpy()  # (the zero lag is the powers' sum over their number)
    want = (raw.to(torch.int64) ** 2).sum((0, 2, 3)).numpy()
    bias = float(((got - want) / want).mean())
    print("mean error of the zero lags", bias, file=sys.stderr, flush=True)
    assert abs(bias) < 2e-8
