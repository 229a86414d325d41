"""Which kernels a call launches, on how many workgroups and with how much LDS.

Every form of a step gives the same bits, so the results do not tell which one
ran; these tests read the launches.
"""
import pytest

from launch_trace import launches
from paper_0708_4182_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0708_4182_amd import lbm as L
    L.load_library()
    return L


def case(nx, ny, storage=0, rounding=0, collision=0):
    c = I.random_channel_case(nx=nx, ny=ny, seed=nx + ny)
    c.params = c.params.replace(storage=storage, rounding=rounding, collision=collision)
    return c


def test_rectangles_leave_room_for_other_handles(lbm):
    """A rectangle launch asks for the LDS its tile needs (phi and, with two steps,
    eight planes of 16 rows of 64 nodes at most: 37.5 KB in FP32), a quarter of a
    compute unit's 160 KB, also where few workgroups would fill the chip."""
    for nx, ny in ((128, 64), (1024, 128)):
        sim = lbm.from_case(case(nx, ny))
        for kernel in ("fused", "two"):
            sim.set_kernel(kernel)
            for l in launches(lambda: sim.step(2)):
                assert l.kernel.startswith("k_node<") and l.lds <= 40 * 1024, l
    b = lbm.Batch([case(256, 80), case(256, 160)])
    b.set_kernel("two")
    for l in launches(lambda: b.step(2)):
        assert l.kernel.startswith("k_batch_node<") and l.lds <= 40 * 1024, l


def test_batch_launches_one_workgroup_per_rectangle(lbm):
    """One long channel beside small ones: 62 x 6 or 62 x 14 node rectangles of one
    step, 58 x 2 or 58 x 10 of two, and at most seven idle workgroups (a multiple
    of the 8 XCDs)."""
    shapes = [(4096, 256)] + [(64, 32)] * 20
    b = lbm.Batch([case(nx, ny) for nx, ny in shapes])
    for kernel, cols, rows in (("fused", 62, 14), ("two", 58, 10)):
        b.set_kernel(kernel)
        tiles = sum(-(-nx // cols) * -(-ny // rows) for nx, ny in shapes)
        (l,) = launches(lambda: b.step(1 if kernel == "fused" else 2))
        assert l.kernel.startswith("k_batch_node<") and tiles <= l.groups < tiles + 8, (l, tiles)
