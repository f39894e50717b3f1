"""The exact gain's own sets, which stay on the device between calls, on a fake HIP runtime: its launches
note whether the sets are clear when a level's voxels are gathered into them."""
import os

import pytest

from tests.fake_runtime import check


@pytest.fixture(scope="module", autouse=True)
def library():
    from paper_2609_40297_amd import mg
    if not os.path.exists(mg.LIB_PATH):
        from paper_2609_40297_amd import build
        build.build()


CALLS = {"own yaw": "mg.mg_eval_exact_marginal(t, g, y, stream=0)",
         "given windows": "mg.mg_eval_exact(t, y, g, xs, a, stream=0)",
         "given windows, rays only": "mg.mg_eval_exact(t, y, g, stream=0)"}


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("level", [1, 2])
def test_sets_are_clear_after_a_call_that_failed(call, level):
    """A call whose merge launch fails leaves voxels in the sets: the next call does not count them."""
    check(f"""
m = new_map()
t = new_tree(m, 30)
g, xs, a, y = Out(64), Out(64), Out(64), Out(64, np.int32)
{CALLS[call]}
F.fake_fail_kernel(b"k_exact_merge", {level})
try:
    {CALLS[call]}
except mg.MGError as e:
    assert e.code == mg.MG_E_DEVICE
else:
    raise AssertionError("the call succeeded")
assert F.fake_dirty() == 0
{CALLS[call]}
assert F.fake_dirty() == 0
""")


def test_trees_share_a_devices_sets():
    """Trees on maps of different sizes take the sets in turn: one allocation per device, as large as the
    largest call needs, freed with the last of these trees."""
    check("""
m, small = new_map((200, 200, 60)), new_map()
g, y = Out(512), Out(512)
big = new_tree(m, 200, star=True)
others = [new_tree(small, n, star=True) for n in (30, 90, 200)] + [new_tree(m, n, star=True) for n in (3, 150)]
mg.mg_eval_exact_marginal(big, g, y, stream=0)
mg.mg_eval_exact(big, y, g, Out(512), Out(512), stream=0)
before = F.fake_live(0)
for t in others + [big]:
    mg.mg_eval_exact(t, y, g, Out(512), Out(512), stream=0)
    mg.mg_eval_exact_marginal(t, g, y, stream=0)
assert F.fake_live(0) == before and F.fake_dirty() == 0
assert F.fake_held(0, 199 * 25 * 25 * 8 * 64) >= 199 * 25 * 25 * 8 * 64
for t in [big] + others[:-1]:
    mg.mg_tree_destroy(t)
held = F.fake_held(0, 199 * 25 * 25 * 8 * 64)
mg.mg_tree_destroy(others[-1])
assert F.fake_held(0, 199 * 25 * 25 * 8 * 64) < held
""")


def test_sets_of_fewer_nodes_where_memory_is_short():
    """Device memory for the sets of a few nodes only: the call takes the level in parts, and the next one
    does not ask for more again."""
    check("""
m = new_map((200, 200, 60))
t = new_tree(m, 200, star=True)
g, xs, a, y = Out(512), Out(512), Out(512), Out(512, np.int32)
F.fake_limit(0, F.fake_live(0) + 5 * 25 * 25 * 8 * 64)
mg.mg_eval_exact(t, y, g, xs, a, stream=0)
before = F.fake_mallocs()
mg.mg_eval_exact(t, y, g, xs, a, stream=0)
mg.mg_eval_exact_marginal(t, g, y, stream=0)
assert F.fake_mallocs() == before and F.fake_dirty() == 0
mg.mg_tree_destroy(t)
t = new_tree(m, 5)
F.fake_limit(0, 1)                                 # (not even one node's)
assert code(mg.mg_eval_exact, t, y, g, xs, a, stream=0) == mg.MG_E_NOMEM
""")


def test_sets_are_clear_after_a_first_call_of_a_larger_tree_that_failed():
    check("""
m = new_map()
g, y = Out(512), Out(512)
t, wide = new_tree(m, 30), new_tree(m, 200, star=True)
mg.mg_eval_exact_marginal(t, g, y, stream=0)
F.fake_fail_kernel(b"k_exact_merge", 1)
assert code(mg.mg_eval_exact, wide, y, g, Out(512), Out(512), stream=0) == mg.MG_E_DEVICE
mg.mg_eval_exact(wide, y, g, Out(512), Out(512), stream=0)
mg.mg_eval_exact_marginal(t, g, y, stream=0)
assert F.fake_dirty() == 0
""")
