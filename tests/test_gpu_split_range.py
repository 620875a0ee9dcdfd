"""FP32 fitness of rows of uneven magnitude (needs an MI355X): layers, units, inputs and
biases of scales far apart, where every operand of the FP16 parts that the register chain
takes has values far below its largest.  Each row is scored through mgfwa_evaluate and held
to FP32's own error: that of the same losses in numpy's float32, against binary64."""
import numpy as np
import pytest

from gpu_util import require_gpu
from oracle import oracle as O
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


def layers(wl, row):
    """Views (W, b) of every layer of a row."""
    at = 0
    for i, o in zip(wl.widths, wl.widths[1:]):
        yield row[at:at + i * o].reshape(o, i), row[at + i * o:at + i * o + o]
        at += i * o + o


_ACT = {"relu": lambda z: np.maximum(z, 0), "identity": lambda z: z, "tanh": np.tanh}


def losses(wl, W, dtype):
    """The losses in numpy: float32 throughout but the mean, or float64."""
    out = []
    for row in W:
        h = wl.x.astype(dtype)
        for i, (w, b) in enumerate(layers(wl, row.astype(dtype))):
            h = h @ w.T + b
            if i < len(wl.acts):
                h = _ACT[wl.acts[i]](h)
        if wl.loss == "mse":
            out.append(((h - wl.y.astype(dtype)) ** 2).astype(np.float64).mean())
        else:
            d = h - h.max(axis=1, keepdims=True)
            l = np.log(np.exp(d).sum(axis=1)) - d[np.arange(len(h)), wl.labels]
            out.append(l.astype(np.float64).mean())
    return np.array(out)


def check(wl, W, what, fit_path=0):
    """Each row to 4 times the error that numpy's float32 makes (sums in another order),
    and 2e-7 for the sum of the losses and the result's own rounding."""
    torch, M = require_gpu()
    g = M.MGFWA(wl.widths, wl.acts, wl.loss, wl.x, wl.y, wl.labels, n_fireworks=2, n_sparks=4,
                n_guiding=2, fit_path=fit_path)
    Wd = torch.zeros((W.shape[0], g.Dp), dtype=torch.float32, device="cuda")
    Wd[:, :wl.dim] = torch.from_numpy(W)
    got = g.evaluate(Wd).cpu().numpy().astype(np.float64)
    g.close()
    want = losses(wl, W, np.float64)
    fp32 = np.abs(losses(wl, W, np.float32) - want)
    err = np.abs(got - want)
    bad = ~(err <= 4 * fp32 + 2e-7 * np.abs(want))
    assert not bad.any(), (what, err[bad] / np.abs(want[bad]), fp32[bad] / np.abs(want[bad]))


def base(widths, act, loss, rows=6, S=700, x_scale=1.0):
    wl = inputs.random_mlp_problem(widths, (act,) * (len(widths) - 2), loss, S, seed=21, x_scale=x_scale)
    W = inputs.random_weights(wl.dim, rows, seed=22, lo=-1.0, hi=1.0)
    for row in W:                       # logits of order one
        for w, b in layers(wl, row):
            w *= np.float32(1.5 / np.sqrt(w.shape[1]))
    return wl, W


CHAIN = [((64, 128, 128, 10), "relu"), ((37, 60, 9), "relu"), ((48, 50, 64, 10), "tanh"),
         ((30, 64, 50, 64, 16), "identity"), ((64, 250, 10), "relu")]


@pytest.mark.parametrize("widths,act", CHAIN)
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_layers_of_different_scale(widths, act, loss):
    wl, W = base(widths, act, loss)
    scales = (1.0, 1e3, 1e5, 1e6, 1e9, 1e12)
    for row, s in zip(W, scales):
        if act == "tanh":
            continue
        parts = list(layers(wl, row))
        parts[0][0][:] *= np.float32(s)
        parts[0][1][:] *= np.float32(s)
        for w, b in parts[1:-1]:
            b *= np.float32(s)
        parts[-1][0][:] *= np.float32(1.0 / s)
    check(wl, W, "layers")


@pytest.mark.parametrize("widths,act", CHAIN)
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_a_large_bias(widths, act, loss):
    """Units switched off (ReLU) or saturated (tanh) by a bias; a unit far above the others
    (identity), whose weights into the next layer are as small."""
    wl, W = base(widths, act, loss)
    for row, s in zip(W, (1e3, 1e5, 1e6, 1e9, 1e12, 1e30)):
        parts = list(layers(wl, row))
        for w, b in parts[:-1]:
            b[3] = np.float32(-s)
        if act == "identity":
            for w, b in parts[1:]:
                w[:, 3] = np.float32(0.5 / s) if s < 1e20 else 0.0
    check(wl, W, "bias")


@pytest.mark.parametrize("widths,act", [c for c in CHAIN if c[1] != "tanh"])
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_units_of_different_scale(widths, act, loss):
    """ReLU and identity commute with a unit's scale: its weights times s, the next layer's
    from it times 1 / s."""
    wl, W = base(widths, act, loss)
    for row, s in zip(W, (1e2, 1e5, 1e7, 1e9, 1e12, 1e15)):
        parts = list(layers(wl, row))
        for (w, b), (wn, _) in zip(parts[:-1], parts[1:]):
            scale = np.ones(len(b), np.float32)
            scale[1::3], scale[2::3] = s, 1.0 / s
            w *= scale[:, None]
            b *= scale
            wn /= scale[None, :]
    check(wl, W, "units")


def test_weights_beyond_the_scales():
    """Weights of 2^80 before and behind a small layer."""
    wl, W = base((40, 60, 50, 9), "relu", "mse", rows=3)
    for row, big in zip(W, (0, 1, 2)):
        for l, (w, b) in enumerate(layers(wl, row)):
            w *= np.float32(2.0 ** 80 if l == big else 2.0 ** -40)
            b *= np.float32(2.0 ** -40 if l == 0 else 1.0)
    check(wl, W, "beyond")


@pytest.mark.parametrize("widths,act", CHAIN)
def test_small_inputs(widths, act):
    """Inputs of s with first-layer weights of 1 / s; and, where the activation commutes
    with it, everything behind them at the scale of s too."""
    for s in (1e-3, 1e-6, 1e-8, 1e-10, 1e-12, 1e-25):
        wl, W = base(widths, act, "mse", rows=2, S=300, x_scale=s)
        w = next(layers(wl, W[0]))[0]
        w *= np.float32(1.0 / s)
        if act != "tanh" and s > 1e-15:
            wl.y *= np.float32(s)
            for _, b in layers(wl, W[1]):
                b *= np.float32(s)
        check(wl, W, f"inputs of {s}")


@pytest.mark.parametrize("widths,act", CHAIN)
@pytest.mark.parametrize("loss", ["ce", "mse"])
def test_inputs_of_different_scale(widths, act, loss):
    """Features of scales far apart, the weights on them as far the other way; and samples
    that have only their small features."""
    for s in (1e2, 1e5, 1e9, 1e12):
        wl, W = base(widths, act, loss, rows=2, S=300)
        scale = np.ones(widths[0], np.float32)
        scale[1::3], scale[2::3] = s, 1.0 / s
        wl.x *= scale
        for row in W:
            next(layers(wl, row))[0][:] /= scale
        wl.x[5::7, 1::3] = 0.0
        check(wl, W, f"features {s}")
