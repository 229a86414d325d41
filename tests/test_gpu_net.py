"""GPU tests of the warm-start network kernels (lbm_net_* through the C ABI).

Forward outputs, the loss and the gradient of every layer are compared with the
plain FP64 network of the oracle (oracle/cnn.py, itself pinned to finite
differences and a brute-force convolution), norm-wise relative error per
output and per parameter block:
  - FP32 activations: <= 1e-5;
  - bf16 activations: <= 3 x the rms error of Monte Carlo arithmetic samples
    of a bf16 network (oracle.cnn.mca_gradient: weights, stored activations
    and layer gradients each with an independent relative error uniform on
    [-2^-8, 2^-8]), and never below 1e-5.  The bars come from that error
    model, computed on the same inputs, not from measured GPU values.
Shapes are chosen ragged: channel counts that are not multiples of the 8 x 16
channel tiles and coarse levels smaller than one 8 x 32 pixel tile.
"""
import numpy as np
import pytest

import oracle.cnn as CNN

pytestmark = pytest.mark.gpu

SMALL = dict(H=16, W=64, chans=(12, 20, 24, 16))


@pytest.fixture(scope="module")
def net():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0708_4182_amd import net as N
    N.load_library()
    return N


def problem(H, W, n, chans, seed):
    """Random inputs, targets, a fluid mask with walls and He-initialised params."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((n, 3, H, W))
    x[:, 0] = rng.random((n, H, W)) < 0.2
    t = rng.standard_normal((n, 3, H, W))
    fluid = rng.random((n, H, W)) > 0.25
    specs = CNN.layer_specs(3, 3, chans)
    theta = CNN.init_params(specs, seed)
    # nonzero biases so that the bias paths are exercised
    o = 0
    for _, ci, co, k in specs:
        o += co * ci * k * k
        theta[o:o + co] = 0.05 * rng.standard_normal(co)
        o += co
    theta = theta.astype(np.float32).astype(np.float64)
    return x.astype(np.float32), t.astype(np.float32), fluid.astype(np.uint8), specs, theta


def to_dev(*arrs):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]


def layer_errors(a, b, specs):
    """Norm-wise relative error of every weight and bias block."""
    out, o = {}, 0
    for name, ci, co, k in specs:
        for part, n in (("W", co * ci * k * k), ("b", co)):
            ref = b[o:o + n]
            out[f"{name}.{part}"] = np.linalg.norm(a[o:o + n] - ref) / max(np.linalg.norm(ref), 1e-30)
            o += n
    return out


def mca_bars(theta, specs, x, t, fluid, samples, seed=0):
    """Bars of a bf16 build against the FP64 network: 3 x the rms over
    ``samples`` Monte Carlo arithmetic samples of the relative error of the
    output ("y"), the loss ("loss") and every parameter block; at least 1e-5."""
    args = (theta, specs, x.astype(np.float64), t.astype(np.float64), fluid.astype(bool))
    L0, g0, y0 = CNN.backward(*args, with_output=True)
    rng = np.random.default_rng(seed)
    ey, el, eg = [], [], []
    for _ in range(samples):
        y, L, g = CNN.mca_gradient(*args, rng)
        ey.append(np.linalg.norm(y - y0) / np.linalg.norm(y0))
        el.append(abs(L - L0) / L0)
        eg.append(layer_errors(g, g0, specs))
    rms = lambda v: float(np.sqrt(np.mean(np.square(v))))
    bars = {"y": max(3 * rms(ey), 1e-5), "loss": max(3 * rms(el), 1e-5)}
    for k in eg[0]:
        bars[k] = max(3 * rms([e[k] for e in eg]), 1e-5)
    return bars, (y0, L0, g0)


def check_against_fp64(m, bf16, x, t, fluid, specs, theta, samples=4, forward_only=False):
    """Run the GPU network and compare output, loss and gradient with the FP64
    network; returns the errors and bars for printing."""
    xd, td, fd = to_dev(x, t, fluid)
    y = m.forward(xd).cpu().numpy()
    if bf16:
        bars, (y0, L0, g0) = mca_bars(theta, specs, x, t, fluid, samples)
    else:
        args = (theta, specs, x.astype(np.float64), t.astype(np.float64), fluid.astype(bool))
        L0, g0, y0 = CNN.backward(*args, with_output=True)
        bars = None
    err = {"y": np.linalg.norm(y - y0) / np.linalg.norm(y0)}
    if not forward_only:
        loss, g = m.gradient(xd, td, fd)
        err["loss"] = abs(loss - L0) / L0
        err.update(layer_errors(g.astype(np.float64), g0, specs))
    if bars is None:
        bars = {k: 1e-5 for k in err}
    over = {k: (err[k], bars[k]) for k in err if not err[k] <= bars[k]}
    worst = max(err, key=lambda k: err[k] / bars[k])
    print(f"bf16={bf16}: forward {err['y']:.3e} (bar {bars['y']:.3e}); "
          f"worst {worst} {err[worst]:.3e} (bar {bars[worst]:.3e})")
    assert not over, over
    return y, err, bars


@pytest.mark.parametrize("bf16", [False, True])
def test_forward_matches_oracle(net, bf16):
    x, t, fluid, specs, theta = problem(n=3, seed=1, **SMALL)
    m = net.Net(SMALL["H"], SMALL["W"], 3, chans=SMALL["chans"], act_bf16=bf16)
    m.set_params(theta)
    y, _, _ = check_against_fp64(m, bf16, x, t, fluid, specs, theta, samples=6, forward_only=True)
    # fewer samples than the batch: same values for those samples
    (xd,) = to_dev(x)
    y2 = m.forward(xd[:1].contiguous()).cpu().numpy()
    np.testing.assert_array_equal(y2[0], y[0])


@pytest.mark.parametrize("bf16", [False, True])
def test_gradient_matches_oracle(net, bf16):
    x, t, fluid, specs, theta = problem(n=2, seed=2, **SMALL)
    m = net.Net(SMALL["H"], SMALL["W"], 2, chans=SMALL["chans"], act_bf16=bf16)
    m.set_params(theta)
    check_against_fp64(m, bf16, x, t, fluid, specs, theta, samples=6)


# channel counts above 32 (the 64-channel output tile of the matrix-core
# convolution; SMALL runs the 32-channel one), ragged against both tiles
WIDE = dict(H=16, W=64, chans=(12, 40, 48, 36))


@pytest.mark.parametrize("bf16", [False, True])
def test_wide_channels_match_oracle(net, bf16):
    """Seed 26 keeps every pre-activation at least 1.6e-5 of its layer's rms
    away from zero (the oracle finds that).  With seed 7 one lies at 1.4e-8 rms,
    FP32 and FP64 put it on different sides of the ReLU, and the gradient of
    the 2 x 8 bottom layers moves by 1.3e-2 (two samples of 16 pixels there)."""
    x, t, fluid, specs, theta = problem(n=2, seed=26, **WIDE)
    m = net.Net(WIDE["H"], WIDE["W"], 2, chans=WIDE["chans"], act_bf16=bf16)
    m.set_params(theta)
    check_against_fp64(m, bf16, x, t, fluid, specs, theta, samples=6)


# Widths that are not multiples of 8 below the top level (40, 20, 10, 5
# columns; 3 rows at the bottom): the convolutions' gather staging and
# per-element stores, and the scalar forms of the ReLU mask and the
# upsampling, which the other shapes (whole 8-pixel groups) do not reach.
RAGGED = dict(H=24, W=40, chans=(8, 12, 16, 8))


@pytest.mark.parametrize("bf16", [False, True])
def test_ragged_widths_match_oracle(net, bf16):
    """Seed 40 keeps every pre-activation at least 5.6e-5 of its layer's rms
    away from zero (the oracle finds that)."""
    x, t, fluid, specs, theta = problem(n=2, seed=40, **RAGGED)
    m = net.Net(RAGGED["H"], RAGGED["W"], 2, chans=RAGGED["chans"], act_bf16=bf16)
    m.set_params(theta)
    check_against_fp64(m, bf16, x, t, fluid, specs, theta, samples=6)


@pytest.mark.parametrize("H,W,chans", [(64, 64, (32, 64, 128, 128)), (24, 40, (12, 40, 48, 36)), (16, 96, (17, 33, 130, 20)),
                                       (40, 264, (32, 64, 128, 128))])
def test_small_batches_are_bitwise_large(net, H, W, chans):
    """One sample runs the small-launch convolution (2 x 32 pixels of 16
    channels per workgroup) where 96 samples run the 8-row tiles: the same bits
    of every output, with cin below, at and above 32 and 128, channel counts that
    fill no tile, vector and plain staging, and H that ends inside a tile."""
    x, _, _, _, theta = problem(H, W, 96, chans, 5)
    big, one = net.Net(H, W, 96, chans=chans), net.Net(H, W, 1, chans=chans)
    for m in (big, one):
        m.set_params(theta.astype(np.float32))
    xd, = to_dev(x)
    ref = big.forward(xd).cpu().numpy()
    for i in (0, 1, 50, 95):
        np.testing.assert_array_equal(one.forward(xd[i:i + 1].contiguous()).cpu().numpy()[0], ref[i])


@pytest.mark.parametrize("H,W,n", [(16, 64, 1), (24, 128, 3), (8, 192, 2), (40, 256, 2), (16, 72, 5)])
def test_gradient_rolls_with_its_inputs(net, H, W, n):
    """Rows are periodic: inputs rolled by a multiple of 8 pixels (the coarsest
    level's pixel) give the same stored activations and layer gradients, rolled,
    so the weight gradient changes only by the order of its FP32 sums (bar
    1e-5 per block, as for FP32).  64- and 32-column and gathered tiles of the
    weight gradient, rows of one and several tiles, H within a tile."""
    chans = (12, 33, 40, 20)
    x, t, fluid, specs, theta = problem(H, W, n, chans, 11)
    m = net.Net(H, W, n, chans=chans)
    m.set_params(theta)
    loss, g = m.gradient(*to_dev(x, t, fluid))
    for shift in (8, 24, W // 2 // 8 * 8, W - 8):
        l2, g2 = m.gradient(*to_dev(*(np.roll(a, shift, axis=-1) for a in (x, t, fluid))))
        assert abs(l2 - loss) <= 1e-12 * abs(loss)
        o = 0
        for _, ci, co, k in specs:
            for size in (co * ci * k * k, co):
                a, b = g[o:o + size].astype(np.float64), g2[o:o + size].astype(np.float64)
                assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(a), (shift, ci, co, size)
                o += size


def test_gradient_is_deterministic(net):
    x, t, fluid, specs, theta = problem(n=2, seed=3, **SMALL)
    m = net.Net(SMALL["H"], SMALL["W"], 2, chans=SMALL["chans"])
    m.set_params(theta)
    d = to_dev(x, t, fluid)
    l1, g1 = m.gradient(*d)
    l2, g2 = m.gradient(*d)
    assert l1 == l2
    np.testing.assert_array_equal(g1, g2)


def test_full_size_matches_oracle(net):
    """The warm-start configuration itself (64 x 256, channels 32/64/128/128),
    one sample, FP32 activations.

    At this size about 40 pre-activations lie within 1e-5 rms of zero (the
    oracle counts them below), closer than the FP32 rounding of a 1152- to
    2304-term sum, so FP32 takes the other ReLU branch at a few of them.  The
    forward output is continuous across such a flip and keeps the 1e-5 bar, as
    does the output layer's gradient, which no flip reaches; the gradient of a
    layer at or below a flipped node moves by about 1e-4 (bar: 1e-3).  The
    small ragged cases above have no such node and hold 1e-5 on every layer."""
    H, W, chans = 64, 256, (32, 64, 128, 128)
    x, t, fluid, specs, theta = problem(H, W, 1, chans, seed=4)
    m = net.Net(H, W, 1, chans=chans, act_bf16=False)
    m.set_params(theta)
    d = to_dev(x, t, fluid)
    y = m.forward(d[0]).cpu().numpy()
    loss, g = m.gradient(*d)
    x64 = x.astype(np.float64)
    y_ref, cache = CNN.forward(theta, specs, x64, keep=True)
    ambiguous = sum(int((np.abs(z) < 1e-5 * np.sqrt((z ** 2).mean())).sum())
                    for name, *_ in specs[:-1] for z in [cache[name][1]])
    e_fwd = np.linalg.norm(y - y_ref) / np.linalg.norm(y_ref)
    ref_loss, ref_g = CNN.backward(theta, specs, x64, t.astype(np.float64), fluid.astype(bool))
    errs = layer_errors(g.astype(np.float64), ref_g, specs)
    worst = max(errs, key=errs.get)
    print(f"full-size forward {e_fwd:.3e}, ambiguous ReLU decisions {ambiguous}, "
          f"gradient worst {worst} {errs[worst]:.3e}, out.W {errs['out.W']:.3e}")
    print("  " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()))
    assert e_fwd <= 1e-5
    assert abs(loss - ref_loss) <= 1e-5 * ref_loss
    assert errs["out.W"] <= 1e-5 and errs["out.b"] <= 1e-5
    assert errs[worst] <= 1e-3, errs


def test_full_size_bf16_matches_oracle(net):
    """The production build (bf16 activations) at the warm-start configuration
    (64 x 256, channels 32/64/128/128), two samples, against the plain FP64
    network with the bars of the bf16 error model (four samples)."""
    H, W, chans = 64, 256, (32, 64, 128, 128)
    x, t, fluid, specs, theta = problem(H, W, 2, chans, seed=14)
    m = net.Net(H, W, 2, chans=chans, act_bf16=True)
    m.set_params(theta)
    _, err, bars = check_against_fp64(m, True, x, t, fluid, specs, theta, samples=4)
    print("  " + " ".join(f"{k}={v:.1e}/{bars[k]:.1e}" for k, v in err.items()))


def test_adam_step_matches_oracle(net):
    x, t, fluid, specs, theta = problem(n=2, seed=5, **SMALL)
    m = net.Net(SMALL["H"], SMALL["W"], 2, chans=SMALL["chans"])
    m.set_params(theta)
    d = to_dev(x, t, fluid)
    th = theta.astype(np.float32).astype(np.float64)
    mo = np.zeros_like(th)
    vo = np.zeros_like(th)
    for step in (1, 2, 3):
        _, g = m.gradient(*d)
        m.adam(lr=1e-3)
        th, mo, vo = CNN.adam(th, g.astype(np.float64), mo, vo, step, lr=1e-3)
        got = m.get_params().astype(np.float64)
        np.testing.assert_allclose(got, th, rtol=1e-6, atol=1e-7)
        th = got


def test_packed_weights_follow_parameter_updates(net):
    """The bf16 build keeps its forward weights packed between calls: after
    lbm_net_set_params and after an Adam step the forward must equal that of
    a new network given the same parameters, bit for bit."""
    x, t, fluid, specs, theta = problem(n=2, seed=9, **SMALL)
    theta2 = problem(n=2, seed=10, **SMALL)[4]
    d = to_dev(x, t, fluid)
    mk = lambda th: (lambda m: (m.set_params(th), m)[1])(net.Net(SMALL["H"], SMALL["W"], 2, chans=SMALL["chans"],
                                                                 act_bf16=True))
    m = mk(theta)
    y1 = m.forward(d[0]).cpu().numpy()
    m.set_params(theta2)
    y2 = m.forward(d[0]).cpu().numpy()
    assert not np.array_equal(y1, y2)
    np.testing.assert_array_equal(y2, mk(theta2).forward(d[0]).cpu().numpy())
    m.train_step(*d, lr=1e-3)
    y3 = m.forward(d[0]).cpu().numpy()
    assert not np.array_equal(y2, y3)
    np.testing.assert_array_equal(y3, mk(m.get_params().astype(np.float64)).forward(d[0]).cpu().numpy())


def test_training_reduces_the_loss(net):
    """Fit a fixed small batch: the loss must fall well below its start."""
    x, t, fluid, specs, theta = problem(n=4, seed=6, **SMALL)
    t = (0.5 * x[:, :1] + 0.1).repeat(3, axis=1).astype(np.float32)
    m = net.Net(SMALL["H"], SMALL["W"], 4, chans=SMALL["chans"])
    m.set_params(theta)
    d = to_dev(x, t, fluid)
    first = m.train_step(*d, lr=2e-3)
    for _ in range(150):
        last = m.train_step(*d, lr=2e-3)
    print(f"loss {first:.4e} -> {last:.4e}")
    assert np.isfinite(last) and last < 0.2 * first


def test_invalid_calls(net):
    import torch
    from paper_0708_4182_amd import lbm
    m = net.Net(16, 64, 2, chans=SMALL["chans"])
    x = torch.zeros((3, 3, 16, 64), device="cuda")
    y = torch.empty((3, 3, 16, 64), device="cuda")
    with pytest.raises(ValueError):                      # the binding: more samples than the batch
        m.forward(x)
    with pytest.raises(ValueError):                      # the binding: wrong width
        m.forward(torch.zeros((1, 3, 16, 32), device="cuda"))
    assert m.lib.lbm_net_forward(m.h, x.data_ptr(), y.data_ptr(), 3) == -1     # the C ABI, before launching
    assert m.lib.lbm_net_forward(m.h, None, y.data_ptr(), 1) == -1
    with pytest.raises(lbm.LBMError, match="ESTATE"):
        m.adam()
    with pytest.raises(ValueError):
        m.set_params(np.zeros(5, np.float32))
