"""Dense read-back of a map's states: rows of every alignment (8-, 4- and 1-byte pieces), runs of bricks
that end inside the grid, and output buffers that start at odd addresses; and the marks of 16-voxel blocks
where the grid's blocks are not a multiple of what a wave takes."""
import numpy as np
import pytest

from paper_2609_40297_amd import workloads as W
from tests.gpu_util import log
from tests.test_gpu_maps import _expected_marks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_40297_amd import mg as mgmod
    mgmod.lib()
    return mgmod


@pytest.mark.parametrize("dims", [(256, 9, 8), (264, 8, 17), (260, 7, 3), (257, 3, 9), (255, 16, 2), (7, 5, 3), (2049, 2, 2)])
@pytest.mark.parametrize("offset", [0, 4, 1])
def test_read_back(mg, dims, offset):
    import torch
    rng = np.random.Generator(np.random.PCG64(sum(dims)))
    st = rng.integers(0, 3, dims[::-1]).astype(np.uint8)
    M = mg.Map(st, 1.0, (0.0, 0.0, 0.0))
    out = torch.full((st.size + 16,), 7, dtype=torch.uint8, device="cuda")
    mg.mg_map_read(M.handle, out[offset:])
    torch.cuda.synchronize()
    log(f"[read] {dims} at +{offset}")
    got = out.cpu().numpy()
    assert np.array_equal(got[offset:offset + st.size], st.reshape(-1))
    assert (got[:offset] == 7).all() and (got[offset + st.size:] == 7).all()      # nothing beside the map is written
    M.close()


@pytest.mark.parametrize("dims", [(16, 16, 16), (48, 16, 48), (80, 47, 33), (15, 64, 64), (144, 32, 16)])
def test_marks_of_blocks(mg, dims):
    rng = np.random.Generator(np.random.PCG64(sum(dims)))
    nb = [-(-d // 16) for d in dims[::-1]]
    st = rng.choice(np.array([W.UNK, W.FREE], np.uint8), nb)
    for a in range(3):
        st = np.repeat(st, 16, a)
    st = np.ascontiguousarray(st[:dims[2], :dims[1], :dims[0]])
    st[rng.uniform(size=st.shape) < 1e-4] = W.OCC
    M = mg.Map(st, 1.0, (0.0, 0.0, 0.0))
    assert np.array_equal(M.read_marked().cpu().numpy(), _expected_marks(st))
    M.close()


@pytest.mark.parametrize("dims", [(129, 127, 48), (257, 176, 190), (260, 121, 100), (264, 100, 72)])
def test_read_back_of_larger_grids(mg, dims):
    """Workgroups of 4, 32, 16 and 8 bricks (the most that leave the chip full), rows of odd and even widths."""
    rng = np.random.Generator(np.random.PCG64(sum(dims)))
    st = rng.integers(0, 3, dims[::-1]).astype(np.uint8)
    M = mg.Map(st, 1.0, (0.0, 0.0, 0.0))
    log(f"[read] {dims}")
    assert np.array_equal(M.read().cpu().numpy(), st)
    M.close()
