"""The step blocks of a pass launch: whether a step waits for its tile's items
or walks them itself, on one item per block or several (a bounded grid), on
contiguous or packed tiles, alone or beside other launches, a call returns the
same bits."""
import threading

import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2606_31098_amd._abi import FLAG_NO_STEP_WAIT as NO_STEP_WAIT
from synth import frames as S

pytestmark = pytest.mark.gpu

LEVELS = ((30, 40, 16), (60, 80, 32), (60, 80, 64))
KEYS = ("poses", "cost", "iterations", "status", "alpha", "best")


def lb(n):
    return max(int(n), 1).bit_length() - 1


def frame(seed, N, M, levels=LEVELS, iters=(4, 3, 3), keep=0):
    f = S.make_frame(2, 0, N=N, M=M, level_shapes=levels, iters=iters[:len(levels)], dsm_side=128, seed=seed)
    f.keep_top, f.prune_level = keep, 0
    return f


def tiles(path, f, dtype, G, ppg, grid, variants, pack):
    with open(path, "a") as fh:
        for L, v in zip(f.levels, variants):
            fh.write(f"C{L.C}_d{int(dtype == 'bf16')}_N{lb(len(L.x))}_M{lb(f.M)}_P{lb(L.H * L.W)}_v3 {G} {ppg} {grid} {v} {pack}\n")
    return str(path)


def same(a, b):
    return all(np.array_equal(a[k], b[k], equal_nan=k in ("cost", "alpha", "poses")) for k in KEYS)


# variants by level: 2 has no step blocks, so that a level with them follows
# one with them directly and over a level without
@pytest.mark.parametrize("dtype,G,variants", [("f32", 4, (3, 3, 3)), ("f32", 8, (4, 2, 4)), ("f32", 16, (1, 1, 1)),
                                              ("bf16", 4, (9, 9, 9)), ("bf16", 16, (10, 2, 10)), ("bf16", 8, (1, 4, 3))])
def test_steps_that_do_not_wait_solve_the_same(tmp_path, dtype, G, variants):
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    M = 2 * G + 3
    N = (ncu // 3 + 9) * (256 // G) - 5             # three hypothesis tiles: more items than one grid of CUs
    assert 3 * ((N + 256 // G - 1) // (256 // G)) > ncu
    f = frame(61, N, M, keep=M - 2)
    d = DeviceFrame(f, dtype=dtype)
    poses = torch.as_tensor(f.poses, device="cuda")
    want = lin = None
    for grid, pack, flags in ((0, 0, 0), (1, 0, 0), (1, 2, 0), (0, 0, NO_STEP_WAIT), (1, 2, NO_STEP_WAIT)):
        path = tmp_path / f"t{grid}{pack}{flags}.txt"
        ctx = Context(0, tune_cache=tiles(path, f, dtype, G, 1, grid, variants, pack), flags=flags)
        assert f"G={G} PPG=1" in ctx.tile_choice(16, int(dtype == "bf16"), N, M, 1200)
        say(f"step wait: {dtype} G={G} variants={variants} grid={grid} pack={pack} flags={flags} N={N} M={M}")
        got = [ctx.solve([d])[0].numpy() for _ in range(3)]            # the graph's capture and two replays
        got_lin = [[t.cpu().numpy() for t in ctx.linearize(d, l, poses)] for l in range(3)]
        ctx.close()
        want, lin = want or got[0], lin or got_lin
        assert (want["status"] == 4).sum() == 2 and (want["status"] < 3).sum() == M - 2
        assert all(same(g, want) for g in got), (grid, pack, flags)
        assert all(np.array_equal(x, y) for a, b in zip(lin, got_lin) for x, y in zip(a, b)), (grid, pack, flags)


def test_steps_that_do_not_wait_serve_and_batch_the_same(tmp_path):
    """Uneven frames in several launch classes: one call (forked launches), the
    static solve, and the serving steps, where frames of one to three levels
    share launches and come and go."""
    from paper_2606_31098_amd.pilot import Context, DeviceFrame, DeviceResult
    fr = [frame(71, 900, 21), frame(72, 500, 9, LEVELS[:1]), frame(73, 700, 40, LEVELS[:2]), frame(74, 2100, 90, keep=30)]
    path = tmp_path / "t.txt"
    for f, (variant, G) in zip(fr, ((3, 4), (4, 8), (1, 16), (4, 4))):
        tiles(path, f, "f32", G, 2, 0, (variant,) * 3, 0)
    dfs = [DeviceFrame(f) for f in fr]
    ctx = Context(0, tune_cache=str(path))
    want = [ctx.solve([d])[0].numpy() for d in dfs]
    ctx.close()
    for flags in (0, NO_STEP_WAIT):
        say(f"step wait: batch, static and serving, flags={flags}")
        ctx = Context(0, tune_cache=str(path), flags=flags, max_slots=3)
        got = [r.numpy() for r in ctx.solve(dfs)]
        assert all(same(a, b) for a, b in zip(got, want)), flags
        got = [r.numpy() for r in ctx.solve_static(dfs)]
        assert all(same(a, b) for a, b in zip(got, want)), flags
        for order in ((0, 1, 2, 3), (3, 1, 0, 2, 1)):
            waiting, live, res = list(order), {}, {}
            for _ in range(400):
                while waiting and len(live) < 3:
                    i = waiting.pop(0)
                    r = DeviceResult(dfs[i].M)
                    live[ctx.admit(dfs[i], r)] = (i, r)
                if not live:
                    break
                ctx.step()
                for slot in [s for s in live if ctx.poll(s)]:
                    i, r = live.pop(slot)
                    res[i] = r.numpy()
            assert sorted(res) == sorted(set(order))
            assert all(same(res[i], want[i]) for i in res), (flags, order)
        ctx.close()


def test_long_launches_wait_for_their_items():
    """A pass of many milliseconds, whose XCDs end one or two apart: the step
    blocks of the early ones have to wait, rather than walk their tiles alone one
    item after the other (this pass then took 30 ms instead of 18)."""
    from paper_2606_31098_amd.pilot import Context, DeviceFrame
    M, ms = 2048, {}
    ctx = Context(0)
    for N in (4000, 40000):                         # neither is sorted
        f = S.make_frame(2, 0, N=N, M=M, level_shapes=((480, 640, 128),), iters=(1,), dsm_side=448, seed=3)
        d = DeviceFrame(f)
        assert "G=8 PPG=16" in ctx.tile_choice(128, 0, N, M, 480 * 640)
        poses = torch.as_tensor(f.poses, device="cuda")
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ctx.linearize(d, 0, poses)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        ms[N] = best
    ctx.close()
    say(f"long launches: {ms}")
    assert ms[40000] < 1.35 * 10 * ms[4000], ms


def test_large_solves_on_two_streams_at_once():
    """Two contexts, each on its own thread and stream, with 1024 hypothesis
    tiles a pass: more step blocks than an XCD holds blocks of both."""
    from paper_2606_31098_amd.pilot import Context, DeviceFrame, DeviceResult
    sets = []
    for seed in (81, 82):
        f = frame(seed, 260, 4096, LEVELS[:2], (3, 2))
        stream = torch.cuda.Stream()
        d = DeviceFrame(f)
        torch.cuda.synchronize()
        ctx = Context(0, stream=stream)
        assert "G=4" in ctx.tile_choice(16, 0, 260, 4096, 1200)
        want = ctx.solve([d])[0]
        stream.synchronize()
        sets.append((ctx, stream, d, want.numpy(), [DeviceResult(d.M) for _ in range(6)]))
    torch.cuda.synchronize()
    say("two threads, six solves each")
    errors = []

    def work(ctx, stream, d, want, results):
        try:
            for r in results:
                ctx.solve([d], [r])
            stream.synchronize()
        except Exception as e:                      # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=s) for s in sets]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for ctx, stream, d, want, results in sets:
        assert all(same(r.numpy(), want) for r in results)
        ctx.close()
