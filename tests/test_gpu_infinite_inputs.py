"""An infinite input that the first layer's activation bounds (needs an MI355X): the loss is
finite, however many units the kernels that stage weights of any activation in LDS pad a
layer with (their zero weights times the infinity are NaNs)."""
import numpy as np
import pytest

from gpu_util import assert_fitness_close, require_gpu
from oracle import oracle as O
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,acts", [
    ((17, 48, 64, 3), ("tanh", "identity")), ((17, 40, 33, 20, 3), ("relu", "identity", "tanh")),
    ((30, 71, 71, 2), ("tanh", "gelu")), ((9, 200, 2), ("tanh",)),
    ((9, 20, 20, 20, 2), ("relu",) * 3), ((33, 50, 40, 60, 3), ("relu",) * 3), ((20, 100, 110, 97, 2), ("relu",) * 3),
    ((40, 60, 9), ("relu",)), ((20, 100, 33, 100, 4), ("tanh", "relu", "tanh"))])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("rows", [3, 300])
def test_an_infinite_input_that_is_bounded(widths, acts, precision, rows):
    """Every first unit sees -inf from the sample (tanh: -1, ReLU: 0).  FP32 to its tolerance;
    BF16 rounds weights and activations to 2^-9, each layer both: within 2^-5 of the loss."""
    torch, M = require_gpu()
    wl = inputs.random_mlp_problem(widths, acts, "mse", 70, seed=8)
    f = widths[0] // 2
    wl.x[33, f] = np.inf
    W = inputs.random_weights(wl.dim, rows, seed=9, lo=-1.0, hi=1.0)
    W[:, f:widths[0] * widths[1]:widths[0]] = -0.5
    at = 0
    for i, o in zip(widths, widths[1:]):
        W[:, at:at + i * o] *= np.float32(1.0 / np.sqrt(i))
        at += i * o + o
    g = M.MGFWA(wl.widths, wl.acts, wl.loss, wl.x, wl.y, wl.labels, n_fireworks=2, n_sparks=4, n_guiding=2,
                precision=precision)
    Wd = torch.zeros((rows, g.Dp), dtype=torch.float32, device="cuda")
    Wd[:, :wl.dim] = torch.from_numpy(W)
    got = g.evaluate(Wd).cpu().numpy()
    g.close()
    want = O.Problem.from_workload(wl).loss_rows(W)
    assert np.isfinite(want).all()
    if precision == "fp32":
        assert_fitness_close(got, want, f"{widths} {acts}")
    else:
        assert np.isfinite(got).all() and (np.abs(got - want) <= 2.0 ** -5 * want).all(), (got, want)
