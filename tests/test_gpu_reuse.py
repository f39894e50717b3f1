"""Device blocks, sensor tables and launch plans outlive the trees they were made for: trees of changing
sizes uploaded, evaluated into new buffers and dropped one after another (and from two threads on their
own streams) give the results of a first, fresh evaluation."""
import threading

import numpy as np
import pytest

from paper_2609_40297_amd import workloads as W
from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_40297_amd import mg as mgmod
    mgmod.lib()
    return mgmod


def _jobs():
    w = W.make("tiny")
    t = w.trees[0]
    wide = W.Sensor(n_az=96, n_el=17, fov_h_deg=60.0, fov_v_deg=50.0, range_m=4.0, yaw_bins=24)
    return w, [(W.Tree(t.pos_m[:n], t.parent[:n]), s) for n, s in
               ((20, w.sensor), (3, w.sensor), (11, wide), (1, wide), (19, w.sensor), (20, wide))]


def _one(mg, M, tree, sensor, stream=None):
    T = mg.Tree(M, tree.pos_m, tree.parent, sensor, stream=stream)
    g, y, d = mg.eval_batch([T], depth=True, stream=stream)
    (stream or __import__("torch").cuda.current_stream()).synchronize()
    out = [v.cpu().numpy().copy() for v in (g, y, d)]
    T.close()
    return out


@pytest.mark.parametrize("threads", [1, 2])
def test_reused_blocks_give_fresh_results(mg, threads):
    import torch
    w, jobs = _jobs()
    M = mg.Map(w.map.states, w.map.voxel_m, w.map.origin_m)
    fresh = [_one(mg, M, t, s) for t, s in jobs]
    bad = []

    def work(seed):
        rng = np.random.Generator(np.random.PCG64(seed))
        stream = torch.cuda.Stream() if threads > 1 else None
        with torch.cuda.stream(stream) if stream else torch.cuda.stream(torch.cuda.current_stream()):
            for k in rng.integers(0, len(jobs), 25):
                got = _one(mg, M, *jobs[k], stream=stream)
                if any(a.tobytes() != b.tobytes() for a, b in zip(got, fresh[k])):
                    bad.append(int(k))

    log(f"[reuse] {threads} thread(s)")
    ts = [threading.Thread(target=work, args=(s,)) for s in range(threads)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad
    M.close()


def test_a_plan_takes_every_call_its_own_buffers(mg):
    """One tree list evaluated into new output buffers on every call, the earlier ones still held."""
    import torch
    w, jobs = _jobs()
    M = mg.Map(w.map.states, w.map.voxel_m, w.map.origin_m)
    trees = [mg.Tree(M, t.pos_m, t.parent, s) for t, s in jobs if s is w.sensor]
    held = [mg.eval_batch(trees, depth=k % 2 == 0) for k in range(5)]
    torch.cuda.synchronize()
    for g, y, d in held[1:]:
        assert torch.equal(g, held[0][0]) and torch.equal(y, held[0][1])
        assert d is None or d.cpu().numpy().tobytes() == held[0][2].cpu().numpy().tobytes()
    for T in trees:
        T.close()
    M.close()


@pytest.mark.parametrize("counts", [(303,), (304,), (101, 101, 101), (102, 101, 101), (1,), (1, 1, 1, 1)])
def test_batches_around_the_smallest_split_over_streams(mg, counts):
    """Batches just below and above the work (304 nodes of this sensor) at which a plan's levels are split
    over streams, of one tree and of several: the same gains and windows as tree by tree."""
    import torch
    w = W.make("step")
    t = w.trees[0]
    m = mg.Map(w.map.states, w.map.voxel_m, w.map.origin_m)
    trees = [mg.Tree(m, t.pos_m[:n], t.parent[:n], w.sensor) for n in counts]
    g, y, _ = mg.eval_batch(trees)
    torch.cuda.synchronize()
    at = 0
    for n, x in zip(counts, trees):
        rg, ry = x.eval_marginal()[:2]
        torch.cuda.synchronize()
        log(f"[split] {counts}: {n} nodes")
        assert torch.equal(g[at:at + n], rg) and torch.equal(y[at:at + n], ry)
        at += n
    for x in trees:
        x.close()
    m.close()
