"""Top-K pruning: which hypotheses survive, at the edges of the ranking's
blocks (16 hypotheses each), with ties, and in a batch with frames that do
not prune."""
import numpy as np
import pytest

from gpu_common import say
from synth import frames as S

pytestmark = pytest.mark.gpu

PRUNED = 4
LEVELS = ((30, 40, 16), (60, 80, 32))


def frame(M, keep, seed=5):
    f = S.make_frame(2, 0, N=300, M=M, level_shapes=LEVELS, iters=(2, 2), dsm_side=96, seed=seed)
    if M > 4:                                   # ties: hypotheses with the same start end at the same cost
        f.poses[M // 2:M // 2 + 2] = f.poses[1]
    f.keep_top, f.prune_level = keep, 0
    return f


@pytest.mark.parametrize("M,keep", [(1, 1), (15, 4), (16, 16), (17, 1), (33, 40), (257, 31), (1100, 128)])
def test_survivors_are_the_lowest_costs(M, keep):
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    say(f"pruning {M} hypotheses to {keep}")
    f = frame(M, keep)
    coarse = frame(M, 0)
    coarse.levels = coarse.levels[:1]           # the costs the ranking sees
    plain = frame(M, 0, seed=6)
    ctx = Context(0)
    # the range prior's ray goes through the finest level's intrinsics: off in
    # all three, so that the one-level frame has the same coarse objective
    for x in (f, coarse, plain):
        x.use_range = 0
    c = ctx.solve([DeviceFrame(coarse)])[0].numpy()
    r, p = [x.numpy() for x in ctx.solve([DeviceFrame(f), DeviceFrame(plain)])]
    order = np.lexsort((np.arange(M), c["cost"]))
    want = np.ones(M, bool)
    want[order[:keep]] = False
    assert (c["status"] != 3).all()
    assert np.array_equal(r["status"] == PRUNED, want)
    assert np.array_equal(r["cost"][want], c["cost"][want])
    assert np.array_equal(r["poses"][want], c["poses"][want])
    assert (p["status"] != PRUNED).all()
