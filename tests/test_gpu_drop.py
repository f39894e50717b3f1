"""Trees dropped while the device still works. In a capture of relaxed mode: the capture goes on, its
replays give the captured evaluation's results, and the dropped tree's memory serves later trees. With
its evaluations still queued: they give their results, whatever trees come next, on any stream."""
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


@pytest.mark.parametrize("planned", [False, True])
def test_drop_during_a_relaxed_capture(mg, planned):
    import torch
    w = W.make("tiny")
    t = w.trees[0]
    M = mg.Map(w.map.states, w.map.voxel_m, w.map.origin_m)
    kept, dropped = (mg.Tree(M, t.pos_m, t.parent, w.sensor) for _ in range(2))
    ref, ref_yaw, _ = kept.eval_marginal()
    if planned:
        mg.eval_batch([dropped])
    else:
        dropped.eval_marginal()
    torch.cuda.synchronize()
    gain, yaw, _ = kept.outputs()
    log(f"[capture] planned={planned}")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        mg.mg_eval_marginal(kept.handle, gain, yaw)
        dropped.close()
    for k in range(4):
        gain.fill_(-1)
        yaw.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(gain, ref) and torch.equal(yaw, ref_yaw), k
        other = mg.Tree(M, t.pos_m, t.parent, w.sensor)       # (eager work between the replays)
        assert torch.equal(mg.eval_batch([other])[0], ref)
        torch.cuda.synchronize()
        other.close()
    kept.close()
    M.close()


def test_drop_with_evaluations_queued(mg):
    """Trees evaluated several times on one stream and dropped without a wait, each followed by the upload
    and evaluation of another tree on a second stream, into memory that the first may still use."""
    import torch
    w = W.make("step")
    t = w.trees[0]
    M = mg.Map(w.map.states, w.map.voxel_m, w.map.origin_m)
    sizes = (500, 470, 455)
    ref = {}
    for n in sizes:
        T = mg.Tree(M, t.pos_m[:n], t.parent[:n], w.sensor)
        ref[n] = [v.clone() for v in T.eval_marginal(depth=True)]
        torch.cuda.synchronize()
        T.close()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = []
    for k in range(12):
        s, n = streams[k % 2], sizes[k % 3]
        with torch.cuda.stream(s):
            T = mg.Tree(M, t.pos_m[:n], t.parent[:n], w.sensor, stream=s)
            for _ in range(3):
                outs.append((n, T.eval_marginal(depth=True, stream=s)))
            outs.append((n, mg.eval_batch([T], depth=True, stream=s)))
            T.close()
    torch.cuda.synchronize()
    log(f"[drop] {len(outs)} evaluations")
    for n, got in outs:
        for a, b in zip(got, ref[n]):
            assert a.reshape(-1).view(torch.int32).equal(b.reshape(-1).view(torch.int32)), n
    M.close()
