"""The LM steps in the last blocks of the pass launch: the sums of a tile's
records at the edges of their batches (R = 64 / G partial sums per column,
eight items each loaded at once), one and two storing waves per item, items
walked one per block and by a bounded grid; linearisations and a solve
against the FP64 oracle at the FP32 bar."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import (NEQ_TOL, POSE_TOL_DEG, POSE_TOL_M, compare_solutions, mask_edges, rel_frobenius, say,
                        unpack_h21)
from synth import frames as S

pytestmark = pytest.mark.gpu


def floor_log2(n):
    return int(n).bit_length() - 1


@pytest.mark.parametrize("G,items,grid", [(4, 1, 0), (4, 17, 0), (4, 129, 2), (8, 8, 0), (8, 9, 0), (8, 65, 0),
                                          (16, 4, 0), (16, 33, 2)])
def test_tile_sums_at_batch_edges_match_oracle(tmp_path, G, items, grid):
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    per = 256 // G                                   # anchors per item (one per lane group)
    N, M = per * items - 3, 2 * G + 1                # ragged last item, ragged last tile
    f = S.make_frame(2, 0, N=N, M=M, level_shapes=((60, 80, 16),), iters=(4,), dsm_side=256, seed=21)
    L = f.levels[0]
    cache = tmp_path / "tune.txt"
    cache.write_text(f"C16_d0_N{floor_log2(N)}_M{floor_log2(M)}_P{floor_log2(L.H * L.W)}_v3 {G} 1 {grid} 3 0\n")
    ctx = Context(0, tune_cache=str(cache))
    assert f"G={G} PPG=1" in ctx.tile_choice(16, 0, N, M, L.H * L.W)
    rng = np.random.default_rng(2)
    poses = np.stack([oracle.compose(oracle.se3_exp(np.concatenate([rng.normal(0, 2, 3), rng.normal(0, 0.02, 3)])),
                                     f.gt_pose) for _ in range(M)])
    say(f"steps: G={G} items={items} grid={grid} N={N} M={M}")
    gpu = ctx.solve([DeviceFrame(f)])[0].numpy()
    rows, fails = compare_solutions(f, gpu, oracle.solve(f, threads=8), POSE_TOL_M, POSE_TOL_DEG)
    assert not fails, fails
    mask_edges(f, poses)
    H21, g, cost, n = ctx.linearize(DeviceFrame(f), 0, torch.as_tensor(poses, device="cuda"))
    torch.cuda.synchronize()
    H, g, cost, n = unpack_h21(H21.cpu().numpy()), g.cpu().numpy(), cost.cpu().numpy(), n.cpu().numpy()
    of = oracle.OracleFrame(f)
    for m in range(M):
        Ho, go, co, no = oracle.linearize(of, 0, poses[m])
        err = rel_frobenius(np.concatenate([H[m], g[m][:, None]], 1), np.concatenate([Ho, go[:, None]], 1))
        assert err <= NEQ_TOL, (m, err)
        assert abs(cost[m] - co) <= 1e-9 * abs(co) and n[m] == no, (m, cost[m], co, n[m], no)


@pytest.mark.parametrize("C", [32, 64, 128])
@pytest.mark.parametrize("G", [4, 8, 16])
@pytest.mark.parametrize("variant", [1, 4])
def test_groups_that_share_projections_with_most_anchors_unseen_match_oracle(tmp_path, variant, G, C):
    """A lane group reads its hypotheses' cells from each other's lanes: poses
    turned so far that some hypotheses see few anchors or none, beside some
    that see all, in tiles whose last one is ragged."""
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    N, M = 517, G + 3
    f = S.make_frame(2, 0, N=N, M=M, level_shapes=((60, 80, C),), iters=(2,), dsm_side=256, seed=31)
    L = f.levels[0]
    cache = tmp_path / "tune.txt"
    cache.write_text(f"C{C}_d0_N{floor_log2(N)}_M{floor_log2(M)}_P{floor_log2(L.H * L.W)}_v3 {G} 2 0 {variant} 0\n")
    ctx = Context(0, tune_cache=str(cache))
    assert f"G={G} PPG=2" in ctx.tile_choice(C, 0, N, M, L.H * L.W)
    turns = [0.0, 0.3, 0.6, np.pi]                   # all seen, some, few, behind the camera
    poses = np.stack([oracle.compose(oracle.se3_exp(np.array([0.1 * m, 0, 0, 0, turns[m % 4], 0])), f.gt_pose)
                      for m in range(M)])
    mask_edges(f, poses)
    say(f"unseen: variant={variant} G={G} C={C}")
    H21, g, cost, n = ctx.linearize(DeviceFrame(f), 0, torch.as_tensor(poses, device="cuda"))
    torch.cuda.synchronize()
    H, g, cost, n = unpack_h21(H21.cpu().numpy()), g.cpu().numpy(), cost.cpu().numpy(), n.cpu().numpy()
    of = oracle.OracleFrame(f)
    for m in range(M):
        Ho, go, co, no = oracle.linearize(of, 0, poses[m])
        assert n[m] == no and abs(cost[m] - co) <= 1e-9 * abs(co), (m, n[m], no, cost[m], co)
        err = rel_frobenius(np.concatenate([H[m], g[m][:, None]], 1), np.concatenate([Ho, go[:, None]], 1))
        assert err <= NEQ_TOL, (m, err)              # nothing seen: the priors' terms alone
