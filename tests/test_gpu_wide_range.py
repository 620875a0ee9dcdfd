"""The wide fitness kernel's FP32 path where rows and samples are of uneven magnitude (needs
an MI355X): what the FP16 parts do not hold to FP32's last bit goes through FP32
instructions, a row or a tile of 256 samples at a time.  Rows are held to FP32's own error,
as in test_gpu_split_range."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_2501_03944_amd import inputs
from test_gpu_split_range import base, check, layers, losses

pytestmark = pytest.mark.gpu

# 127 inputs: the fewest columns (128 with the bias) that take the parts
WIDE = [((127, 33, 3), "relu"), ((200, 256, 16), "tanh"), ((161, 64, 2), "identity"), ((784, 130, 10), "relu")]


@pytest.mark.parametrize("widths,act", WIDE)
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_a_large_bias(widths, act, loss):
    """Units switched off (ReLU) or saturated (tanh) by a bias; a unit far above the others
    (identity), whose weights into the next layer are as small."""
    wl, W = base(widths, act, loss)
    for row, s in zip(W, (1e3, 1e5, 1e6, 1e9, 1e12, 1e30)):
        parts = list(layers(wl, row))
        parts[0][1][3] = np.float32(-s)
        if act == "identity":
            parts[1][0][:, 3] = np.float32(0.5 / s) if s < 1e20 else 0.0
    check(wl, W, "bias", fit_path=2)


@pytest.mark.parametrize("widths,act", [c for c in WIDE if c[1] != "tanh"])
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_units_and_layers_of_different_scale(widths, act, loss):
    wl, W = base(widths, act, loss)
    for i, (row, s) in enumerate(zip(W, (1.0, 1e2, 1e5, 1e9, 1e12, 1e18))):
        (w, b), (w2, _) = layers(wl, row)
        scale = np.full(len(b), s, np.float32)
        if i % 2:
            scale[1::3], scale[2::3] = 1.0, 1.0 / s
        w *= scale[:, None]
        b *= scale
        w2 /= scale[None, :]
    check(wl, W, "units", fit_path=2)


def test_weights_beyond_the_scales():
    """First-layer weights of 2^80 and 2^-80, second-layer ones that undo it; and no weights."""
    wl, W = base((140, 70, 9), "relu", "mse", rows=4)
    for row, s in zip(W, (2.0 ** 80, 2.0 ** -80, 2.0 ** -20, 0.0)):
        (w, b), (w2, _) = layers(wl, row)
        w *= np.float32(s)
        b *= np.float32(s)
        w2 *= np.float32(1.0 / s if s else 1.0)
    check(wl, W, "beyond", fit_path=2)


@pytest.mark.parametrize("widths,act", WIDE)
def test_small_inputs(widths, act):
    for s in (1e-3, 1e-8, 1e-10, 1e-12, 1e-25):
        wl, W = base(widths, act, "mse", rows=2, S=300, x_scale=s)
        w = next(layers(wl, W[0]))[0]
        w *= np.float32(1.0 / s)
        if act != "tanh" and s > 1e-15:
            wl.y *= np.float32(s)
            for _, b in layers(wl, W[1]):
                b *= np.float32(s)
        check(wl, W, f"inputs of {s}", fit_path=2)


@pytest.mark.parametrize("widths,act", WIDE)
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_inputs_of_different_scale(widths, act, loss):
    """Features of scales far apart, the weights on them as far the other way, in all tiles
    of samples or in one; beside rows that the parts hold."""
    for s in (1e2, 1e5, 1e9, 1e12):
        for one_tile in (False, True):
            wl, W = base(widths, act, loss, rows=3, S=600)
            scale = np.ones(widths[0], np.float32)
            scale[1::3], scale[2::3] = s, 1.0 / s
            at = slice(256, 512, 5) if one_tile else slice(0, 600)
            wl.x[at] *= scale
            next(layers(wl, W[1]))[0][:] /= scale
            wl.x[5::7, 1::3] = 0.0
            check(wl, W, f"features {s} {one_tile}", fit_path=2)


@pytest.mark.parametrize("lag", [False, True])
@pytest.mark.parametrize("scale", [1.0, 1e-6])
def test_sparks_of_a_wide_box(lag, scale):
    """A generation of sparks that all but equal their fireworks, whose first layers lie far
    below the box: rows that their own exponent holds, and rows with one weight or bias of
    the box's size; then one of sparks that the box's exponent holds, in the same rows."""
    torch, M = require_gpu()
    widths, N, lam = (150, 40, 4), 4, 8
    wl, W = base(widths, "relu", "mse", rows=N, S=300)
    wl.x[:, 77] = 0.0
    for row in W:
        (w, b), (w2, _) = layers(wl, row)
        w *= np.float32(scale)
        b *= np.float32(scale)
        w2 /= np.float32(scale)
    W[1, 77] = 3e8                       # on the feature that is zero
    W[2, 150 * 40 + 5] = -9e8            # bias of unit 5
    plain = inputs.random_weights(wl.dim, N, seed=3, lo=-9e8, hi=9e8)
    for row in plain:                    # (its losses are to be FP32 values)
        next(reversed(list(layers(wl, row))))[0][:] *= np.float32(1e-9)
    g = M.MGFWA(wl.widths, wl.acts, wl.loss, wl.x, wl.y, wl.labels, n_fireworks=N, n_sparks=lam,
                n_guiding=2, lb=-1e9, ub=1e9, fit_path=2, seed=4, lag_guiding=lag, loser_out=False)
    for rows, amp in ((W, scale * 1e-9), (plain, 1e-9), (W, scale * 1e-9)):
        st = g.state()
        torch.cuda.synchronize()
        st["F"][:, :wl.dim] = torch.from_numpy(rows).cuda()
        st["A"].fill_(amp)
        torch.cuda.synchronize()
        g.step(1)
        got = g.state_numpy()["Yc"].reshape(N, -1)[:, :lam].astype(np.float64)
        want = losses(wl, rows, np.float64)
        # (a spark's weights are within 1e-9 of their scale of its firework's: far within 1e-5)
        err = np.abs(got - want[:, None])
        assert (err <= 1e-5 * want[:, None]).all(), (err / want[:, None])
    g.close()


def test_an_infinite_feature_costs_a_tile():
    """One infinite feature in 32 tiles of samples: its tile runs on FP32 instructions, at a
    third of the rate; twice the time is far above that."""
    torch, M = require_gpu()
    wl = inputs.random_mlp_problem((784, 256, 10), ("relu",), "ce", 8192, seed=8)
    ms = {}
    for infinite in (False, True):
        x = wl.x.copy()
        if infinite:
            x[3000, 1] = -np.inf
        g = M.MGFWA(wl.widths, wl.acts, wl.loss, x, wl.y, wl.labels, n_fireworks=2, n_sparks=4, n_guiding=2)
        W = torch.zeros((512, g.Dp), dtype=torch.float32, device="cuda")
        W[:, :wl.dim] = torch.from_numpy(inputs.random_weights(wl.dim, 512, seed=9, lo=-1.0, hi=1.0)).cuda()
        best = np.inf
        for _ in range(4):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            t0.record()
            g.evaluate(W)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1))
        ms[infinite] = best
        g.close()
    assert ms[True] < 2.0 * ms[False], ms
