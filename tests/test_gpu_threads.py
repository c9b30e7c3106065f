"""Plans of different LDS sizes called from several threads at once, each on a stream of its own: the same bytes as one
after another."""

import math
import sys
import threading

import pytest
import torch

import paper_0909_0001_amd as omni

pytestmark = pytest.mark.gpu

# line kernels and grouped inverses of 8 to 160 KiB, and a grid of the runtime-shape kernel
LEVELS = [[[6, 6]], [[5, 3], [3, 3], [3, 3]], [[16, 16]], [[3, 17], [8, 5]]]


def test_plans_on_threads():
    F, T, calls = 2, 20, 30
    gen = torch.Generator().manual_seed(1)
    plans, raws, want = [], [], []
    for lv in LEVELS:
        N = math.prod(n for l in lv for n in l)
        raws.append(torch.randint(-127, 128, (T, F, N, 2), generator=gen, dtype=torch.int16).to(torch.int8).cuda())
        plans.append(omni.Plan(lv, None, F, "ci8", "fp32"))
        want.append(plans[-1].correlate(raws[-1]).clone())
    torch.cuda.synchronize()
    print("threads", LEVELS, file=sys.stderr, flush=True)
    bad = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(calls):
                    got = plans[i].correlate(raws[i])
                    torch.cuda.current_stream().synchronize()
                    if not torch.equal(got, want[i]):
                        bad.append(LEVELS[i])
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # (a thread's error would be lost)
            bad.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(LEVELS))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
