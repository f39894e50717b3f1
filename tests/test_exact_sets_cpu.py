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
