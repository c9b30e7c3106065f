"""The inverse of arrays beyond the caches, axis by axis with a thread a line, against the same cells inverted in
groups of axes (a plan of one channel, whose arrays are small)."""

import pytest
import torch

import paper_0909_0001_amd as omni

pytestmark = pytest.mark.gpu

# levels, channels: at least 2^25 cells; first axes of 32 and 32, and of 8, 8, 16 and 16
CASES = [([(16, 16), (8, 8)], 129), ([(4, 4), (8, 8), (4, 4)], 32)]


@pytest.mark.parametrize("levels,F", CASES)
def test_line_inverse_matches_groups(levels, F):
    n = 1
    for x, y in levels:
        n *= x * y
    gen = torch.Generator().manual_seed(5)
    raw = torch.randint(-127, 128, (1, F, n, 2), generator=gen, dtype=torch.int16).to(torch.int8).cuda()
    got = omni.Plan(levels, nchan=F, dtype="ci8").correlate(raw)
    one = omni.Plan(levels, nchan=1, dtype="ci8")
    for f in (0, F // 2, F - 1):
        want = one.correlate(raw[:, f : f + 1].contiguous())[0].to(torch.complex128)
        # one sample: the cells are the same; every pass' stored float32 values add at most 2^-24 of the array's
        # norm, six passes on one side and three on the other: 9 x 6e-8
        err = (got[f].to(torch.complex128) - want).norm() / want.norm()
        print(f"{levels} channel {f}: {err:.2e}", flush=True)
        assert err < 6e-7
