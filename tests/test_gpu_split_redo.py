"""Samples that the FP32 register chain's FP16 parts cannot hold (needs an MI355X): values
that are not finite go the way that IEEE arithmetic sends them, whatever else the data
holds, and a few such samples cost little more than a few samples."""
import dataclasses

import numpy as np
import pytest

from gpu_util import assert_fitness_close, require_gpu
from oracle import oracle as O
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


def _job(wl, x):
    torch, M = require_gpu()
    return torch, M.MGFWA(wl.widths, wl.acts, wl.loss, x, wl.y, wl.labels, n_fireworks=2, n_sparks=4,
                          n_guiding=2, fit_path=1)


def _evaluate(wl, x, W):
    torch, g = _job(wl, x)
    Wd = torch.zeros((W.shape[0], g.Dp), dtype=torch.float32, device="cuda")
    Wd[:, :wl.dim] = torch.from_numpy(W)
    got = g.evaluate(Wd).cpu().numpy()
    g.close()
    return got


@pytest.mark.parametrize("widths", [(40, 60, 9), (24, 64, 50, 10), (20, 50, 50, 50, 8)])
@pytest.mark.parametrize("S", [70, 5000])
def test_a_sample_does_not_depend_on_others(widths, S):
    """A NaN input is a NaN loss (+inf), and a NaN pre-activation (an infinite weight on a
    feature that is zero) gives one result, with and without an infinite input in another
    sample."""
    acts = ("relu",) * (len(widths) - 2)
    wl = inputs.random_mlp_problem(widths, acts, "mse", S, seed=8)
    W = inputs.random_weights(wl.dim, 4, seed=9, lo=-1.0, hi=1.0)
    W[2, 3] = np.inf                     # unit 0, input 3
    W[:, 11:widths[0] * widths[1]:widths[0]] = -0.5
    got = {}
    for nan_input in (False, True):
        for infinite_input in (False, True):
            x = wl.x.copy()
            x[:, 3] = 0.0
            if infinite_input:
                x[41, 11] = np.inf       # every unit of the first layer is switched off
            if nan_input:
                x[S - 1, 5] = np.nan
            got[nan_input, infinite_input] = f = _evaluate(wl, x, W)
            if nan_input:
                assert np.isinf(f).all(), (infinite_input, f)
            else:
                ref = O.Problem.from_workload(dataclasses.replace(wl, x=x)).loss_rows(W)
                rows = [0, 1, 3]
                assert_fitness_close(f[rows], ref[rows], f"{widths} infinite input {infinite_input}")
    assert np.isinf(got[False, False][2]) == np.isinf(got[False, True][2]), got


@pytest.mark.parametrize("widths,S,rows", [((64, 128, 128, 10), 4096, 256), ((32, 64, 10), 40000, 40)])
def test_an_infinite_feature_costs_a_slab_group(widths, S, rows):
    """One infinite feature in the data set: the fitness takes little longer (a block stages
    the weights once more and runs one slab group again; twice the time is far above that,
    and a block's whole sample range sample by sample is far above twice)."""
    torch, M = require_gpu()
    wl = inputs.random_mlp_problem(widths, ("relu",) * (len(widths) - 2), "ce", S, seed=8)
    ms = {}
    for infinite in (False, True):
        x = wl.x.copy()
        if infinite:
            x[S // 3, 1] = -np.inf
        torch, g = _job(wl, x)
        W = torch.zeros((rows, g.Dp), dtype=torch.float32, device="cuda")
        W[:, :wl.dim] = torch.from_numpy(inputs.random_weights(wl.dim, rows, seed=9, lo=-1.0, hi=1.0)).cuda()
        best = np.inf
        for _ in range(5):
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
