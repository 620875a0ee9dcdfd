"""Cross-entropy of confident networks (needs an MI355X): losses down to FP32's smallest
values, where exponentials below 2^-126 are all that is left of a loss."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


NETS = [((3, 20, 4), 1), ((40, 64, 9), 1), ((64, 128, 128, 10), 0), ((17, 40, 33, 20, 3), 0)]


@pytest.mark.parametrize("widths,fit_path,precision", [(*net, p) for net in NETS for p in ("fp32", "bf16")] +
                         [((150, 40, 4), 2, "fp32")])
def test_losses_below_the_normal_range(widths, fit_path, precision):
    """Logits that are the last biases alone, class 0 ahead of the others by x: the loss is
    log1p((n - 1) e^-x), within 1e-5 of it or two of FP32's smallest steps (the sum over the
    samples and the mean round once each)."""
    torch, M = require_gpu()
    wl = inputs.random_mlp_problem(widths, ("relu",) * (len(widths) - 2), "ce", 64, seed=3)
    wl.labels[:] = 0
    x = np.array([1.0, 40.0, 86.0, 88.0, 92.0, 97.0, 101.0], np.float32)
    W = np.zeros((len(x), wl.dim), np.float32)
    W[:, wl.dim - widths[-1]] = x
    g = M.MGFWA(wl.widths, wl.acts, wl.loss, wl.x, wl.y, wl.labels, n_fireworks=2, n_sparks=4, n_guiding=2,
                fit_path=fit_path, precision=precision)
    Wd = torch.zeros((len(x), g.Dp), dtype=torch.float32, device="cuda")
    Wd[:, :wl.dim] = torch.from_numpy(W)
    got = g.evaluate(Wd).cpu().numpy().astype(np.float64)
    g.close()
    want = np.log1p((widths[-1] - 1) * np.exp(-x.astype(np.float64)))
    tol = 1e-5 * want + 2 * 2.0 ** -149 * (widths[-1] - 1)
    if precision == "bf16":             # (the biases are bfloat16 there: 1, 40, 86 and 88 are)
        got, want, tol = got[:4], want[:4], tol[:4]
    assert (np.abs(got - want) <= tol).all(), (got, want)
