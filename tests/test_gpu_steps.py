"""GPU parity at the edges of the block step of the ray walk: coordinates and parameters near the
largest a grid allows (where the rounding of a position along the ray is largest), rays that start
on voxel faces, edges and corners, and directions along the axes and their diagonals, on maps of
nested uniform blocks, bit for bit against the oracle."""
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


def _blocks(rng, dims):
    """States of nested uniform blocks: 16-voxel blocks of one state, some split down to 8, 4, 2 and 1."""
    nx, ny, nz = dims
    st = np.zeros((nz, ny, nx), np.uint8)
    for edge, keep in ((16, 1.0), (8, 0.4), (4, 0.3), (2, 0.3), (1, 0.2)):
        n = [-(-d // edge) for d in (nz, ny, nx)]
        s = rng.choice(np.array([W.UNK, W.FREE, W.OCC], np.uint8), n, p=[0.45, 0.548, 0.002])
        take = rng.uniform(size=n) < keep
        for a in (0, 1, 2):
            s, take = np.repeat(s, edge, a), np.repeat(take, edge, a)
        s, take = s[:nz, :ny, :nx], take[:nz, :ny, :nx]
        st = np.where(take, s, st)
    return st


@pytest.mark.parametrize("dims, range_vox", [((8192, 17, 16), 9000.0), ((16, 4099, 23), 5000.0), ((9, 16, 2047), 2050.5),
                                             ((63, 65, 33), 70.0), ((63, 65, 33), 64.0)])
def test_block_step_at_the_largest_coordinates(mg, dims, range_vox):
    from oracle import mgref
    rng = np.random.Generator(np.random.PCG64(sum(dims)))
    m = W.Map(states=_blocks(rng, dims), voxel_m=1.0, origin_m=np.zeros(3, np.float32))
    ext = np.array(dims, np.float32)
    n = 12
    pos = (rng.uniform(0.0, 1.0, (n, 3)) * (ext - 0.01)).astype(np.float32)
    pos[1] = np.floor(pos[1])                               # a voxel corner
    pos[2, 0] = np.floor(pos[2, 0])                         # a face
    pos[3, 1:] = np.floor(pos[3, 1:])                       # an edge
    pos[4] = np.floor(pos[4]) + np.float32(0.5)             # a centre
    pos[5] = np.nextafter(ext, np.float32(0))               # the far corner
    pos[6] = 0.0                                            # the near corner
    par = np.array([-1] + [int(rng.integers(0, i)) for i in range(1, n)], np.int32)
    tree = W.Tree(pos_m=pos, parent=par)
    sensor = W.Sensor(n_az=72, n_el=21, fov_h_deg=90.0, fov_v_deg=63.0, range_m=float(range_vox), yaw_bins=8,
                      az_offset_deg=-2.5)                   # column centres on the axes and diagonals, row 10 level
    log(f"[steps] {dims}: {np.bincount(m.states.reshape(-1), minlength=3).tolist()}")
    ref = mgref.eval_tree(m, tree, sensor, n_threads=threads())
    got = gpu_eval_tree(mg, m, tree, sensor, mode="both")
    assert_same(got, ref, keys=("g_db", "k_db", "D", "g_abs", "k_abs"))
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="batch"), ref)


@pytest.mark.parametrize("copies, range_vox", [(1, 64.0), (18, 64.0), (35, 64.0), (69, 64.0), (137, 64.0), (1, 8.0), (1, 7.5),
                                               (35, 0.25)])
def test_split_rays_give_the_rays_results(mg, copies, range_vox):
    """A level of `copies` nodes (the launch takes 8, 8, 4, 2 and 1 lanes a ray): parameters at which a
    ray is split fall on voxel boundaries (ranges 64 and 8, nodes on voxel corners, rays along the axes),
    inside free and unknown blocks and past first hits and the grid's faces; and ranges
    of less than a voxel per lane."""
    from oracle import mgref
    rng = np.random.Generator(np.random.PCG64(40 + copies))
    dims = (61, 66, 40)
    m = W.Map(states=_blocks(rng, dims), voxel_m=1.0, origin_m=np.zeros(3, np.float32))
    pos = (rng.uniform(0.0, 1.0, (copies + 1, 3)) * (np.array(dims) - 0.01)).astype(np.float32)
    pos[1::2] = np.floor(pos[1::2])
    par = np.array([-1] + [0] * copies, np.int32)
    tree = W.Tree(pos_m=pos, parent=par)
    sensor = W.Sensor(n_az=216, n_el=33, fov_h_deg=90.0, fov_v_deg=66.0, range_m=range_vox, yaw_bins=8,
                      az_offset_deg=-(5.0 / 6.0))
    log(f"[split] {copies} nodes below the root")
    ref = mgref.eval_tree(m, tree, sensor, n_threads=threads())
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="both"), ref, keys=("g_db", "k_db", "D", "g_abs", "k_abs"))


@pytest.mark.parametrize("seed", [3, 4])
def test_hits_at_parameter_zero(mg, seed):
    """Nodes on voxel faces, edges and corners beside occupied voxels, and inside them: the first hit at
    parameter 0 keeps the sign of its zero (depth buffers are compared by their bits)."""
    from oracle import mgref
    rng = np.random.Generator(np.random.PCG64(seed))
    dims = (19, 17, 14)
    st = rng.choice(np.array([W.UNK, W.FREE, W.OCC], np.uint8), dims[::-1], p=[0.3, 0.3, 0.4])
    m = W.Map(states=st, voxel_m=1.0, origin_m=np.zeros(3, np.float32))
    pos = (rng.uniform(0.0, 1.0, (40, 3)) * np.array(dims)).astype(np.float32)
    pos = np.where(rng.uniform(size=pos.shape) < 0.7, np.floor(pos), pos).astype(np.float32)
    tree = W.Tree(pos_m=pos, parent=np.array([-1] + [int(rng.integers(0, i)) for i in range(1, 40)], np.int32))
    sensor = W.Sensor(n_az=72, n_el=21, fov_h_deg=90.0, fov_v_deg=63.0, range_m=9.0, yaw_bins=8, az_offset_deg=-2.5)
    ref = mgref.eval_tree(m, tree, sensor, n_threads=threads())
    zeros = ref["D"] == 0.0
    log(f"[zero hits] {int(zeros.sum())} of {zeros.size}, {int(np.signbit(ref['D'][zeros]).sum())} negative")
    assert 0 < int(np.signbit(ref["D"][zeros]).sum()) < int(zeros.sum())
    assert_same(gpu_eval_tree(mg, m, tree, sensor), ref)
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="batch"), ref)


@pytest.mark.parametrize("n_az, n_el, bins, wide, copies", [(512, 61, 256, 127, 1), (512, 61, 256, 127, 300),
                                                           (512, 61, 256, 1, 700), (432, 33, 144, 70, 40), (3, 1, 3, 1, 5),
                                                           (270, 5, 45, 22, 2)])
def test_window_selection_by_several_workgroups(mg, n_az, n_el, bins, wide, copies):
    """The most bins, windows of one bin and of almost half of them, one tile and 1024 of them, whole and
    partial ones, selected by 4, 3 and 1 workgroups a node: a child of each of `copies` nodes sees what
    its parent's mask, built from the tiles, leaves it."""
    from oracle import mgref
    rng = np.random.Generator(np.random.PCG64(bins + copies))
    dims = (61, 66, 40)
    m = W.Map(states=_blocks(rng, dims), voxel_m=1.0, origin_m=np.zeros(3, np.float32))
    n = 1 + 2 * copies
    pos = (rng.uniform(0.0, 1.0, (n, 3)) * (np.array(dims) - 0.01)).astype(np.float32)
    pos[1 + copies:] = pos[1:1 + copies] + np.float32(0.25)
    pos = np.minimum(pos, np.array(dims, np.float32) - np.float32(0.01))
    par = np.array([-1] + [0] * copies + list(range(1, 1 + copies)), np.int32)
    tree = W.Tree(pos_m=pos, parent=par)
    sensor = W.Sensor(n_az=n_az, n_el=n_el, fov_h_deg=360.0 * wide / bins, fov_v_deg=60.0, range_m=12.0, yaw_bins=bins,
                      az_offset_deg=1.0)
    log(f"[select] {n_az}x{n_el}, {bins} bins, {copies} nodes")
    ref = mgref.eval_tree(m, tree, sensor, n_threads=threads())
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="both"), ref, keys=("g_db", "k_db", "D", "g_abs", "k_abs"))
    assert_same(gpu_eval_tree(mg, m, tree, sensor, mode="batch"), ref)
