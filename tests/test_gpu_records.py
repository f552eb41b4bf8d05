"""A tile whose partial records pass 4 GiB: 2^25 anchors at 16 lanes per anchor
and one anchor per lane group are 2^21 work items of 2 KB each.  All but 2000
anchors lie behind the camera, so the normal equations are those of the 2000
alone (FP64 oracle, the FP32 bar), wherever they stand among the others, and
each of the others adds the constant cost of an anchor out of view."""
import copy

import numpy as np
import pytest
import torch

import oracle
from gpu_common import NEQ_TOL, mask_edges, rel_frobenius, say, unpack_h21
from synth import frames as S

pytestmark = pytest.mark.gpu


def test_records_past_4_gib_are_summed_whole(tmp_path):
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    G, few, M = 16, 2000, 17                         # a full tile and a ragged one
    N = (1 << 25) + 16000 - 3
    f = S.make_frame(2, 0, N=few, M=M, level_shapes=((60, 80, 16),), iters=(2,), dsm_side=256, seed=41)
    L = f.levels[0]
    poses = np.stack([oracle.compose(oracle.se3_exp(np.array([0.2 * m, -0.1 * m, 0.0, 0.0, 0.0, 0.001 * m])), f.gt_pose)
                      for m in range(M)])
    mask_edges(f, poses)
    df = DeviceFrame(f)
    R, t = f.gt_pose[:9].reshape(3, 3), f.gt_pose[9:]
    behind = R.T @ (np.array([0.0, 0.0, -500.0]) - t)
    at = torch.as_tensor(np.linspace(0, N - 1, few).astype(np.int64), device="cuda")
    keep = []
    for name, v, fill in (("x", L.x, behind[0]), ("y", L.y, behind[1]), ("z", L.z, behind[2]), ("ref_w", L.ref_w, 1.0)):
        big = torch.full((N,), float(fill), dtype=torch.float32, device="cuda")
        big[at] = torch.as_tensor(np.ascontiguousarray(v, dtype=np.float32), device="cuda")
        setattr(df.s.level[0], name, big.data_ptr())
        keep.append(big)
    ref = torch.zeros((N, 16), dtype=torch.float32, device="cuda")
    ref[at] = torch.as_tensor(np.ascontiguousarray(L.ref, dtype=np.float32), device="cuda")
    keep.append(ref)
    df.s.level[0].ref = ref.data_ptr()
    df.s.level[0].N = N
    cache = tmp_path / "tune.txt"
    cache.write_text(f"C16_d0_N25_M4_P{(L.H * L.W).bit_length() - 1}_v3 {G} 1 0 3 0\n")
    ctx = Context(0, tune_cache=str(cache))
    assert "G=16 PPG=1" in ctx.tile_choice(16, 0, N, M, L.H * L.W)
    say(f"records: N={N} M={M} G={G}, {2048 * ((N + 15) // 16) / 2 ** 30:.2f} GiB a tile")
    H21, g, cost, n = ctx.linearize(df, 0, torch.as_tensor(poses, device="cuda"))
    torch.cuda.synchronize()
    H, g, cost, n = unpack_h21(H21.cpu().numpy()), g.cpu().numpy(), cost.cpu().numpy(), n.cpu().numpy()
    ctx.close()
    of = oracle.OracleFrame(f)
    fu = copy.deepcopy(f)                            # one more anchor, out of view
    U = fu.levels[0]
    U.x, U.y, U.z = (np.append(v, np.float32(b)) for v, b in zip((U.x, U.y, U.z), behind))
    U.ref, U.ref_w = np.vstack([U.ref, np.zeros((1, 16), np.float32)]), np.append(U.ref_w, np.float32(1.0))
    unseen = oracle.linearize(oracle.OracleFrame(fu), 0, poses[0])[2] - oracle.linearize(of, 0, poses[0])[2]
    for m in range(M):
        Ho, go, co, no = oracle.linearize(of, 0, poses[m])
        co += (N - few) * unseen
        assert n[m] == no, (m, n[m], no)
        err = rel_frobenius(np.concatenate([H[m], g[m][:, None]], 1), np.concatenate([Ho, go[:, None]], 1))
        assert err <= NEQ_TOL, (m, err)
        assert abs(cost[m] - co) <= 1e-9 * abs(co), (m, cost[m], co)
