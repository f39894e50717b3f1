"""Levels just on each side of the sizes at which a trace launch gives a ray to 8, 4, 2 or 1 lanes, per
tree and in a batch, bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2609_40297_amd import workloads as W
from tests.gpu_util import assert_same, gpu_eval_tree, log, threads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_40297_amd import mg as mgmod
    mgmod.lib()
    return mgmod


@pytest.mark.parametrize("copies, lanes", [(16, 8), (17, 4), (32, 4), (33, 2), (65, 2), (66, 1)])
def test_levels_around_the_lane_counts(mg, copies, lanes):
    """A node is 14 x 9 blocks of 16 x 4 rays, a wave each: 16384 waves are 16 nodes at 8 lanes a ray, 32 at
    4 and 65 at 2. The level below the root has `copies` nodes, on voxel corners and off them, and each has
    a child, so that its mask is built from the first hits that the lanes stored."""
    from oracle import mgref
    assert copies * 126 * lanes <= 16384 and (lanes == 8 or copies * 126 * 2 * lanes > 16384)
    rng = np.random.Generator(np.random.PCG64(60 + copies))
    dims = (61, 66, 40)
    nb = [-(-d // 8) for d in dims[::-1]]
    st = rng.choice(np.array([W.UNK, W.FREE], np.uint8), nb)
    for a in range(3):
        st = np.repeat(st, 8, a)
    st = np.ascontiguousarray(st[:dims[2], :dims[1], :dims[0]])
    st[rng.uniform(size=st.shape) < 2e-3] = W.OCC
    m = W.Map(states=st, voxel_m=1.0, origin_m=np.zeros(3, np.float32))
    n = 1 + 2 * copies
    pos = (rng.uniform(0.0, 1.0, (n, 3)) * (np.array(dims) - 1.01)).astype(np.float32)
    pos[1:1 + copies:2] = np.floor(pos[1:1 + copies:2])
    pos[1 + copies:] = pos[1:1 + copies] + np.float32(0.25)
    tree = W.Tree(pos_m=pos, parent=np.array([-1] + [0] * copies + list(range(1, 1 + copies)), np.int32))
    sensor = W.Sensor(n_az=216, n_el=33, fov_h_deg=90.0, fov_v_deg=66.0, range_m=64.0, yaw_bins=8, az_offset_deg=-(5.0 / 6.0))
    log(f"[lanes] {copies} nodes, {lanes} lanes a ray")
    ref = mgref.eval_tree(m, tree, sensor, n_threads=threads())
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="both"), ref, keys=("g_db", "k_db", "D", "g_abs", "k_abs"))
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="batch"), ref)
