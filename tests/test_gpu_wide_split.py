"""The wide fitness kernel's FP32 path in two FP16 parts (needs an MI355X): scales of
samples and weights far from one, infinities, and the error against the oracle's
binary64 loss (rows through mgfwa_evaluate, so each row's exponent is its own)."""
import numpy as np
import pytest

from gpu_util import assert_fitness_close, require_gpu
from oracle import oracle as O
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


def _evaluate(wl, W):
    torch, M = require_gpu()
    g = M.MGFWA(wl.widths, wl.acts, wl.loss, wl.x, wl.y, wl.labels, n_fireworks=2, n_sparks=4,
                n_guiding=2, fit_path=2)
    Wd = torch.zeros((W.shape[0], g.Dp), dtype=torch.float32, device="cuda")
    Wd[:, :wl.dim] = torch.from_numpy(W)
    got = g.evaluate(Wd).cpu().numpy()
    g.close()
    return got


# 127 inputs: the fewest columns (128 with the bias) that take the FP16 parts
@pytest.mark.parametrize("widths,act", [((127, 33, 3), "relu"), ((200, 256, 16), "tanh"),
                                        ((300, 130, 1), "gelu"), ((161, 64, 2), "identity")])
@pytest.mark.parametrize("xs,ws", [(1e-5, 1.0), (1.0, 1e-6), (3e5, 1e-3), (1e8, 2.0), (1.0, 1e4)])
def test_scales(widths, act, xs, ws):
    """Squared error has no cancellation against its own scale: 1e-5 relative (the FP32
    fitness tolerance) whatever the scales of samples and weights."""
    wl = inputs.random_mlp_problem(widths, (act,), "mse", 300, seed=5, x_scale=xs)
    W = inputs.random_weights(wl.dim, 9, seed=6, lo=-ws, hi=ws)
    W[1] *= np.float32(1e-3)              # rows of different scales in one launch
    W[2, ::7] = 0.0
    want = O.Problem.from_workload(wl).loss_rows(W)
    assert_fitness_close(_evaluate(wl, W), want, f"{widths} {act} x {xs} w {ws}", atol=0.0)


@pytest.mark.parametrize("act", ["relu", "tanh", "gelu", "identity"])
def test_infinities(act):
    """An infinite weight, bias or input gives the loss that IEEE arithmetic gives: a
    hidden unit switched off by a bias of -inf, a saturated tanh, +inf elsewhere (NaN
    counts as +inf)."""
    wl = inputs.random_mlp_problem((140, 20, 3), (act,), "mse", 70, seed=8)
    D, in_, hid = wl.dim, 140, 20
    W = inputs.random_weights(D, 6, seed=9, lo=-1.0, hi=1.0)
    W[1, in_ * hid + 4] = -np.inf         # b1 of unit 4
    W[2, in_ * hid + 5] = np.inf
    W[3, 7] = np.inf                      # W1[0][7]
    W[5, in_ * hid:in_ * hid + hid] = -np.inf
    for infinite_input in (False, True):
        if infinite_input:
            wl.x[33, 11] = np.inf
            W[4, 11:in_ * hid:in_] = -0.5  # every unit sees -inf from that sample
        with np.errstate(invalid="ignore"):
            want = O.Problem.from_workload(wl).loss_rows(W)
        want = np.where(np.isnan(want), np.inf, want)
        got = _evaluate(wl, W)
        finite = np.isfinite(want)
        assert np.array_equal(np.isfinite(got), finite), (act, infinite_input, got, want)
        assert_fitness_close(got[finite], want[finite], f"{act} infinite input {infinite_input}")
        if act == "relu":
            assert finite[1] != infinite_input and finite[4]
