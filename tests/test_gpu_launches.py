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


@pytest.mark.parametrize("kernel,tile,form,threads,strips,chunks", [
    ("fused", (256, 0), "k_node<", 512, 5, 22),       # the default: 62 x 6 rectangles
    ("fused", (64, 8), "k_step<", 64, 5, 17), ("fused", (512, 16), "k_step<", 512, 1, 9),
    ("fused", (64, 1), "k_step<", 64, 5, 131), ("fused", (256, 4), "k_step<", 256, 2, 33),
    ("two", (256, 7), "k_stepk<", 256, 2, 19), ("two", (512, 16), "k_stepk<", 512, 1, 9),
    ("three", (256, 5), "k_stepk<", 256, 2, 27)])
def test_tiles_are_marched_as_asked(lbm, kernel, tile, form, threads, strips, chunks):
    """A tile that was asked for is marched in strips of its columns and chunks of
    its rows also on a small lattice; only the default tile leaves the form open."""
    sim = lbm.from_case(case(300, 131))
    sim.set_kernel(kernel)
    sim.set_tile(*tile)
    (l,) = launches(lambda: sim.step({"two": 2, "three": 3}.get(kernel, 1)))
    assert l.kernel.startswith(form) and l.threads == threads, l
    assert strips * chunks <= l.groups < strips * chunks + 8, l


@pytest.mark.parametrize("kernel,tile", [("two", (256, 8)), ("two", (512, 40)), ("three", (256, 0)), ("three", (512, 16))])
def test_steps_left_by_a_multi_step_kernel(lbm, kernel, tile):
    """They take the library's form at any tile."""
    sim = lbm.from_case(case(300, 131))
    sim.set_kernel(kernel)
    sim.set_tile(*tile)
    k = {"two": 2, "three": 3}[kernel]
    ls = launches(lambda: sim.step(2 * k - 1))
    assert [l.kernel.split("<")[0] for l in ls] == ["k_stepk"] + ["k_node"] * (k - 1), ls


@pytest.mark.parametrize("tile,form", [((256, 32), "k_batch_node<"), ((256, 16), "march"), ((64, 8), "march"),
                                       ((128, 32), "march")])
def test_batch_tiles_are_marched_as_asked(lbm, tile, form):
    b = lbm.Batch([case(300, 131), case(64, 40)])
    b.set_tile(*tile)
    for kernel, march in (("fused", "k_batch_tiles<"), ("two", "k_batch_tilesk<")):
        b.set_kernel(kernel)
        (l,) = launches(lambda: b.step(1 if kernel == "fused" else 2))
        assert l.kernel.startswith(march if form == "march" else form), l


def test_autotuners_time_the_march_too(lbm):
    """On a small lattice and a small batch the tuners try low marches beside the
    rectangles."""
    sim = lbm.from_case(case(300, 131))
    ls = launches(lambda: sim.autotune(reps=1))
    assert {(l.kernel.split("<")[0], l.threads) for l in ls} >= {("k_node", 512), ("k_step", 64), ("k_step", 256)}
    assert max(l.groups for l in ls if l.kernel.startswith("k_step<") and l.threads == 64) >= 5 * 33     # 4 rows
    b = lbm.Batch([case(300, 131), case(64, 40)])
    ls = launches(lambda: b.autotune(reps=1))
    assert {l.kernel.split("<")[0] for l in ls} >= {"k_batch_node", "k_batch_tiles", "k_batch_tilesk", "k_batch_step"}


@pytest.mark.parametrize("nx,ny,tall,groups", [(4100, 900, "false", 9 * 56), (5000, 900, "false", 10 * 51),
                                               (4100, 1900, "true", 9 * 28)])
def test_automatic_rows_fill_the_form_that_runs(lbm, nx, ny, tall, groups):
    """FP32 TRT, two steps, 512 columns: two workgroups of the form for low chunks
    are resident per compute unit (256 of them), one of the form for tall chunks;
    automatic rows give one wave of the form they launch."""
    import torch
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    sim = lbm.from_case(case(nx, ny, collision=1))
    sim.set_kernel("two")
    sim.set_tile(512, 0)
    (l,) = launches(lambda: sim.step(2))
    assert l.kernel.startswith("k_stepk<") and l.kernel.endswith(tall + ">"), l
    assert groups <= l.groups < groups + 8, l
