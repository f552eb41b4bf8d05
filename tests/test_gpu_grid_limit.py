"""A launch whose work items alone fit the largest grid (2^24 - 1 blocks of 256
threads), but not with a step block per hypothesis tile behind them."""
import numpy as np
import pytest
import torch

from gpu_common import say
from synth import frames as S

pytestmark = pytest.mark.gpu


def test_items_and_steps_past_the_largest_grid(tmp_path):
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    N, M, G = 1023 * 64, 65536, 4
    assert 1023 * (M // G) < 1 << 24 <= 1024 * (M // G)      # items, items and steps
    f = S.make_frame(2, 0, N=N, M=3, level_shapes=((30, 40, 16),), iters=(1,), dsm_side=384, seed=91)
    away = f.poses[0].copy()
    away[8:12] = (-away[8], away[9], away[10], -away[11] - 1000.0)
    away[6:8] = -away[6:8]                                   # everything behind the camera
    poses = np.tile(away, (M, 1))
    seen = np.array([0, 1, G, M // 2 + 3, M - 1])
    poses[seen] = f.poses[[0, 1, 2, 0, 1]]
    f.poses = poses
    d = DeviceFrame(f)
    out = []
    for ppg in (1, 16):                                      # 16760832 items, and a 16th of them
        cache = tmp_path / f"t{ppg}.txt"
        cache.write_text(f"C16_d0_N15_M16_P10_v3 {G} {ppg} 0 3 0\n")
        ctx = Context(0, tune_cache=str(cache))
        assert f"G={G} PPG={ppg}" in ctx.tile_choice(16, 0, N, M, 1200)
        say(f"grid limit: PPG={ppg}")
        out.append([t.cpu().numpy() for t in ctx.linearize(d, 0, d.poses)])
        ctx.close()
    (H, g, cost, n), (H1, g1, cost1, n1) = out
    assert np.array_equal(n, n1) and (n[seen] > 1000).all() and n.sum() == n[seen].sum()
    # the same pairs in another order: 65472 FP32 terms per sum
    assert np.allclose(H[seen], H1[seen], rtol=0, atol=1e-5 * np.abs(H1[seen]).max())
    assert np.allclose(g[seen], g1[seen], rtol=0, atol=1e-5 * np.abs(g1[seen]).max())
    assert np.allclose(cost, cost1, rtol=1e-12, atol=0)
