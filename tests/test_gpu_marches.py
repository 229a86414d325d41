"""The marches and rectangles that automatic tiles reach only on larger lattices,
asked for by tile or size, bitwise against the one-step march.

Small lattices at automatic rows run rectangles of nodes whatever the kernel, so
the two-step march, its form for tall FP32 chunks and the higher one-step rectangle
are named here: every storage format, rounding mode and operator, on single
lattices and in batches.
"""
import numpy as np
import pytest

from launch_trace import launches
from paper_0708_4182_amd import inputs as I

pytestmark = pytest.mark.gpu

# storage, rounding, collision
MODELS = [(0, 0, 0), (0, 0, 1), (0, 0, 2), (1, 0, 1), (1, 1, 0), (1, 1, 2), (2, 0, 0), (2, 0, 2), (2, 1, 1)]


@pytest.fixture(scope="module")
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0708_4182_amd import lbm as L
    L.load_library()
    return L


def case(nx, ny, storage, rounding, collision):
    c = I.random_channel_case(nx=nx, ny=ny, seed=nx + ny)
    c.params = c.params.replace(storage=storage, rounding=rounding, collision=collision)
    return c


def same(a, b, msg=""):
    for x, y in zip(a.moments(), b.moments()):
        np.testing.assert_array_equal(x, y, err_msg=msg)
    assert a.flux() == b.flux()


@pytest.mark.parametrize("tile", [(256, 7), (256, 17), (256, 33), (512, 12), (512, 40)])
@pytest.mark.parametrize("storage,rounding,collision", MODELS)
def test_two_step_march(lbm, storage, rounding, collision, tile):
    """Low and (32 rows and more: another form in FP32) tall chunks, strips one column
    over and short of whole tiles, odd counts that leave a single step."""
    for nx, ny in ((251, 61), (499, 131)):
        c = case(nx, ny, storage, rounding, collision)
        ref, b = lbm.from_case(c), lbm.from_case(c)
        ref.set_tile(128, 17)
        b.set_kernel("two")
        b.set_tile(*tile)
        for n in (4, 7):
            ref.step(n)
            b.step(n)
            same(ref, b, f"{nx} x {ny} after {ref.steps_done} steps")
    (l,) = launches(lambda: b.step(2))
    tall = storage == 0 and ny // -(-ny // tile[1]) >= 32
    assert l.kernel.startswith("k_stepk<") and l.kernel.endswith(f", 2, {'true' if tall else 'false'}>"), l


@pytest.mark.parametrize("tile", [(256, 16), (256, 33), (512, 40)])
@pytest.mark.parametrize("kernel", ["two", "three"])
@pytest.mark.parametrize("storage,rounding,collision", MODELS)
def test_multi_step_batch_march(lbm, storage, rounding, collision, kernel, tile):
    """The same in a batch of unlike channels, one of them retired on the way."""
    cases = [case(nx, ny, storage, rounding, collision) for nx, ny in ((5, 24), (251, 97), (300, 131), (499, 70))]
    a, b = lbm.Batch(cases), lbm.Batch(cases)
    a.set_tile(128, 17)
    b.set_kernel(kernel)
    b.set_tile(*tile)
    for n in (6, 5):
        a.step(n)
        b.step(n)
        for i in range(len(cases)):
            for x, y in zip(a.moments(i), b.moments(i)):
                np.testing.assert_array_equal(x, y, err_msg=f"channel {i}")
        for x, y in zip(a.flux(), b.flux()):
            np.testing.assert_array_equal(x, y)
        if n == 6:
            for q in (a, b):
                q.retire([i == 1 for i in range(len(cases))])
    (l,) = launches(lambda: b.step({"two": 2, "three": 3}[kernel]))
    tall = storage == 0 and tile[1] >= 32
    assert l.kernel.startswith("k_batch_tilesk<") and l.kernel.endswith("true>" if tall else "false>"), l


@pytest.mark.parametrize("nx,ny", [(1100, 300), (1303, 262)])
@pytest.mark.parametrize("storage,rounding,collision", MODELS)
def test_high_one_step_rectangles(lbm, storage, rounding, collision, nx, ny):
    """More than three 62 x 6 rectangles per compute unit: 62 x 14 ones, also with an
    acceleration field."""
    import torch
    c = case(nx, ny, storage, rounding, collision)
    ref, b = lbm.from_case(c), lbm.from_case(c)
    ref.set_tile(128, 17)

    def steps():
        for n in (3, 6):
            ref.step(n)
            b.step(n)
            same(ref, b)
        (l,) = launches(lambda: b.step(1))
        ref.step(1)
        assert l.kernel.startswith("k_node<") and l.kernel.endswith(", 1, 2>"), l

    steps()
    if rounding or collision:
        return
    acc = torch.from_numpy(1e-5 * np.random.default_rng(nx).standard_normal((2, ny, nx)).astype(np.float32)).cuda()
    for s in (ref, b):
        s.set_accel_field(acc)
    steps()
