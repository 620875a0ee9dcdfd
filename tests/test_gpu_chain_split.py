"""The register-chain fitness kernels in two FP16 parts, and the instances with weights
in LDS and run-time activations (needs an MI355X): every plan at the edges of its row
blocks, scales of samples and weights far from one, and values that are not finite,
against the oracle's binary64 loss (rows through mgfwa_evaluate: each row's exponent is
its own)."""
import numpy as np
import pytest

from gpu_util import assert_fitness_close, require_gpu
from oracle import oracle as O
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


def _evaluate(wl, W):
    torch, M = require_gpu()
    g = M.MGFWA(wl.widths, wl.acts, wl.loss, wl.x, wl.y, wl.labels, n_fireworks=2, n_sparks=4,
                n_guiding=2, fit_path=1)
    Wd = torch.zeros((W.shape[0], g.Dp), dtype=torch.float32, device="cuda")
    Wd[:, :wl.dim] = torch.from_numpy(W)
    got = g.evaluate(Wd).cpu().numpy()
    g.close()
    return got


# widths at and beside the row blocks' edges; 37 inputs end inside a K block, 48 leave
# half of one; 33 samples leave most of the last slab group empty
@pytest.mark.parametrize("widths,acts", [
    ((37, 49, 9), "relu"), ((20, 64, 10), "tanh"), ((48, 255, 16), "relu"), ((20, 113, 8), "gelu"),
    ((37, 65, 64, 11), "relu"), ((30, 128, 128, 10), "tanh"), ((64, 129, 160, 10), "relu"),
    ((37, 48, 20, 33, 15), "gelu"), ((32, 96, 96, 96, 10), "relu"), ((32, 112, 97, 112, 10), "tanh"),
    ((29, 50, 50, 50, 12), "identity"), ((9, 50, 50, 50, 2), "identity")])
@pytest.mark.parametrize("S", [33, 700])
def test_every_plan(widths, acts, S):
    torch, M = require_gpu()
    wl = inputs.random_mlp_problem(widths, (acts,) * (len(widths) - 2), "ce", S, seed=5, x_scale=0.5)
    N, lam = 2, 6
    g = M.MGFWA.from_workload(wl, seed=9, n_fireworks=N, n_sparks=lam, n_guiding=2, max_generations=10)
    plans = len(g.fit_candidates(0))
    before, D = g.state_numpy(), wl.dim
    g.close()
    cfg = O.make_config(N=N, lam=lam, G=2, seed=9, T=10)
    rows = np.stack([O.explosion_row(cfg, before["F"][r // lam, :D], before["A"][r // lam], r, 1)
                     for r in range(N * lam)])
    want = O.Problem.from_workload(wl).loss_rows(rows)
    for i in range(plans):
        g = M.MGFWA.from_workload(wl, seed=9, n_fireworks=N, n_sparks=lam, n_guiding=2,
                                  max_generations=10)
        g.set_fit_plan(0, i)
        info = g.fit_plan(0)
        g.step(1)
        y = g.state_numpy()["Yc"][:, :lam].ravel()
        g.close()
        assert_fitness_close(y, want, f"{widths} {acts} S={S} plan {i} {info['row_blocks']}")


@pytest.mark.parametrize("widths,act", [((37, 60, 9), "relu"), ((20, 200, 8), "tanh"),
                                        ((48, 50, 64, 10), "gelu"), ((30, 64, 64, 64, 16), "identity")])
@pytest.mark.parametrize("xs,ws", [(1e-5, 1.0), (1.0, 1e-6), (3e5, 1e-3), (1e6, 2.0), (1.0, 1e4)])
def test_scales(widths, act, xs, ws):
    """Squared error has no cancellation against its own scale: 1e-5 relative (the FP32
    fitness tolerance) whatever the scales of samples and weights."""
    wl = inputs.random_mlp_problem(widths, (act,) * (len(widths) - 2), "mse", 300, seed=5, x_scale=xs)
    W = inputs.random_weights(wl.dim, 9, seed=6, lo=-ws, hi=ws)
    W[1] *= np.float32(1e-3)              # rows of different scales in one launch
    W[2, ::7] = 0.0
    W[3] = 0.0
    want = O.Problem.from_workload(wl).loss_rows(W)
    got = _evaluate(wl, W)
    fits = want * 300 < 1e38              # the kernels' FP32 sums of the losses overflow beyond it
    assert fits.any()
    assert_fitness_close(got[fits], want[fits], f"{widths} {act} x {xs} w {ws}", atol=0.0)


@pytest.mark.parametrize("act", ["relu", "tanh", "gelu", "identity"])
def test_not_finite(act):
    """An infinite weight, bias, input or activation gives the loss that IEEE arithmetic
    gives (NaN counts as +inf)."""
    in_, hid = 40, 60
    wl = inputs.random_mlp_problem((in_, hid, 9), (act,), "mse", 70, seed=8)
    W = inputs.random_weights(wl.dim, 7, seed=9, lo=-1.0, hi=1.0)
    W[1, in_ * hid + 4] = -np.inf         # b1 of unit 4
    W[2, in_ * hid + 5] = np.inf
    W[3, 7] = np.inf                      # W1[0][7]
    W[5, in_ * hid:in_ * hid + hid] = -np.inf
    W[6, :in_ * hid] *= np.float32(3e38)  # products beyond FP32's range
    for infinite_input in (False, True):
        if infinite_input:
            wl.x[33, 11] = np.inf
            W[4, 11:in_ * hid:in_] = -0.5  # every unit sees -inf from that sample
        p = O.Problem.from_workload(wl)
        with np.errstate(invalid="ignore", over="ignore"):
            want = p.loss_rows(W)
        want = np.where(np.isnan(want), np.inf, want)
        got = _evaluate(wl, W)
        rows = [0, 1, 2, 3, 4, 5]          # (row 6 is finite in binary64: beyond FP32's range there)
        finite = np.isfinite(want)
        assert np.array_equal(np.isfinite(got)[rows], finite[rows]), (act, infinite_input, got, want)
        keep = [r for r in rows if finite[r]]
        assert_fitness_close(got[keep], want[keep], f"{act} infinite input {infinite_input}")
        assert not np.isnan(got).any()
