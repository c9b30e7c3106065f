"""Parity with the oracle on the paths that sides with large prime factors take: the general kernel for runtime shapes
(no register transform), the line kernel's passes of 11 and 13 values, and the inverse's plain sums, staged in LDS where
there are columns for it or not, beside its wide group passes."""

import json
import math
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_0909_0001_amd as omni

pytestmark = pytest.mark.gpu

# levels, format, T, F, forward schedule, and what the inverse's plain sums see (columns of one sum, length m)
CASES = [
    ([[3, 17]], "ci8", 40, 3, "runtime", "untiled"),
    ([[2, 19]], "ci4", 33, 2, "runtime", "untiled"),
    ([[6, 31], [2, 2]], "cf32", 17, 2, "runtime", "untiled"),
    ([[17, 3]], "ci8", 40, 3, "lines", "untiled"),  # a prime first axis is summed directly, divided among work-groups
    ([[19, 2]], "cf32", 33, 2, "lines", "untiled"),
    ([[11, 13]], "ci8", 50, 3, "lines", "groups"),
    ([[13, 12]], "cf32", 29, 2, "lines", "groups"),
    ([[22, 26]], "ci4", 20, 2, "lines", "groups"),
    ([[13, 1], [11, 2]], "ci8", 9, 5, "lines", "groups"),
    ([[2560, 1]], "ci8", 3, 1, "lines", "untiled"),  # m = 5120: longer than a group
    ([[31, 2], [4, 4]], "ci8", 6, 32, "lines", "tiled"),  # the first sum reads the real accumulator, 8192 columns
    ([[34, 4], [4, 4]], "ci8", 5, 8, "lines", "tiled"),  # m = 68: 16 columns a work-group
    ([[4, 4], [4, 17]], "ci4", 5, 24, "runtime", "tiled"),  # the last sum writes the visibilities
    ([[8, 8], [17, 3]], "ci8", 3, 16, "runtime", "tiled"),  # values behind the axis, fewer than a tile's columns
    ([[17, 1]], "cf32", 2, 8200, "runtime", "tiled"),  # one axis: real input, scaled output, a ragged last tile
]


def random_raw(dtype, T, F, N, gen):
    if dtype == "cf32":
        return torch.randn((T, F, N, 2), generator=gen).float()
    if dtype == "ci8":
        return torch.randint(-127, 128, (T, F, N, 2), generator=gen, dtype=torch.int16).to(torch.int8)
    re = torch.randint(-7, 8, (T, F, N), generator=gen, dtype=torch.int16)
    im = torch.randint(-7, 8, (T, F, N), generator=gen, dtype=torch.int16)
    return ((re & 0xF) << 4 | (im & 0xF)).to(torch.uint8)


@pytest.mark.parametrize("levels,dtype,T,F,schedule,inverse", CASES)
def test_odd_sides_match_oracle(levels, dtype, T, F, schedule, inverse):
    dims = [n for lvl in levels for n in lvl]
    N = math.prod(dims)
    gen = torch.Generator().manual_seed(N + T)
    raw = random_raw(dtype, T, F, N, gen)
    print(f"[odd sides] {levels} {dtype} T={T} F={F}: {schedule}, {inverse}", file=sys.stderr, flush=True)
    plan = omni.Plan(levels, None, F, dtype, "fp32")
    a = json.loads(plan.describe())["arrays"][0]
    assert a["kernel"] == "fused_fp32" and a["schedule"] == schedule and a["inverse"] == inverse
    vis = plan.correlate(raw.cuda())
    torch.cuda.synchronize()
    ref = oracle.visibilities(oracle.decode(raw.numpy(), dtype, T, F, N), dims).reshape(F, -1)
    got = vis.cpu().numpy().reshape(F, -1)
    zero = np.abs(ref[:, ref.shape[1] // 2])
    # float32 transforms of at most 5120 values and float32 sums of at most 64 samples: the float32 form's 1e-5
    assert float((np.abs(got - ref).max(axis=1) / zero).max()) <= 1e-5
