"""Pruning frames of thousands of hypotheses, where a block of the ranking takes
several chunks of 16: the survivors, and what a serving step pays for the
ranking's launch while there is nothing to rank."""
import time

import numpy as np
import pytest
import torch

from gpu_common import say
from synth import frames as S

pytestmark = pytest.mark.gpu

PRUNED = 4


def frame(M, keep, iters, seed=5):
    f = S.make_frame(2, 0, N=120, M=M, level_shapes=((30, 40, 16), (60, 80, 32)), iters=iters, dsm_side=96, seed=seed)
    f.poses[M // 2:M // 2 + 2] = f.poses[1]          # ties
    f.keep_top, f.prune_level, f.use_range = keep, 0, 0
    return f


@pytest.mark.parametrize("M,keep", [(2048, 100), (2049, 100), (2065, 1), (8191, 500), (8192, 8192)])
def test_survivors_are_the_lowest_costs(M, keep):
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    say(f"pruning {M} hypotheses to {keep}")
    f, coarse = frame(M, keep, (2, 1)), frame(M, 0, (2, 1))
    coarse.levels = coarse.levels[:1]                # the costs the ranking sees
    ctx = Context(0)
    c = ctx.solve([DeviceFrame(coarse)])[0].numpy()
    r = ctx.solve([DeviceFrame(f)])[0].numpy()
    ctx.close()
    live = c["status"] != 3                          # degenerate ones are not ranked
    order = [m for m in np.lexsort((np.arange(M), c["cost"])) if live[m]]
    want = live.copy()
    want[order[:keep]] = False
    assert np.array_equal(r["status"] == PRUNED, want)
    assert np.array_equal(r["cost"][want], c["cost"][want])


def test_steps_without_a_ranking_are_cheap():
    from paper_2606_31098_amd.pilot import Context, DeviceFrame, DeviceResult
    M, frames, steps = 8192, 4, 8
    cost = {}
    for keep in (0, 64):
        f = frame(M, keep, (60, 1))
        f.lm = dict(f.lm, step_tol_t=0.0, step_tol_r=0.0, cost_tol=0.0)     # all stay at the coarse level
        d = DeviceFrame(f)
        best = 1e9
        for _ in range(4):
            ctx = Context(0, max_slots=64)
            slots = [ctx.admit(d, DeviceResult(M)) for _ in range(frames)]
            assert None not in slots
            ctx.step()
            ctx.sync()
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(steps):
                ctx.step()
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / steps * 1e6)
            ctx.close()
        cost[keep] = best
    say(f"serving step without / with pruning frames: {cost[0]:.0f} / {cost[64]:.0f} us")
    # two launches' worth; a pass over every cost by every block took 45 to 100
    assert cost[64] - cost[0] < 25.0, cost
