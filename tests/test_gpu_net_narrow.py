"""The whole-network kernel of narrow fixed networks (needs an MI355X): at the edges of
its column blocks, chunk groups and rows its values are bit for bit those of the layer
kernels whose sums it takes (the sequential ones under plan 4 against plan 0), and within
FP32's error bound of the oracle with the K-split sums (plan 3)."""
import numpy as np
import pytest

from gpu_util import require_gpu
from oracle import oracle as O
from paper_2501_03944_amd import inputs
from test_gpu_testbed import assert_net_close

pytestmark = pytest.mark.gpu

SEQUENTIAL, K_SPLIT, WHOLE = 0, 3, 4


# widths around the 16-column blocks and the 2 / 4 / 8 chunk variants, uneven layers, one
# to twelve layers; inputs shorter than a chunk, around the groups of 64, and longer than
# one launch takes (512)
@pytest.mark.parametrize("widths,act", [
    ((1, 1), None), ((3, 16, 1), "tanh"), ((63, 17, 1), "gelu"), ((64, 32, 32, 1), "relu"),
    ((65, 33, 64, 1), "relu"), ((129, 64, 16, 64, 1), "gelu"), ((100, 128, 128, 1), "gelu"),
    ((511, 65, 127, 3, 1), "tanh"), ((513, 128, 16, 1), "relu"), ((1030, 1), None), ((700, 20, 1), "identity"),
    ((10,) + (96,) * 11 + (1,), "relu")])
@pytest.mark.parametrize("rows", [(2, 4), (3, 10), (16, 150)], ids=lambda r: str(r[0] * r[1]))
def test_sums_of_the_layer_kernels(widths, act, rows):
    torch, M = require_gpu()
    wl = inputs.net_input_problem(widths, (act,) * (len(widths) - 2), seed=sum(widths))
    N, lam = rows
    got = {}
    for plan in (SEQUENTIAL, K_SPLIT, WHOLE):
        g = M.MGFWA.from_workload(wl, n_fireworks=N, n_sparks=lam, n_guiding=2, max_generations=10, seed=7)
        before = g.state_numpy()
        g.set_fit_plan(0, plan)
        g.step(1)
        got[plan] = g.state_numpy()["Yc"][:, :lam].ravel()
        g.close()
    assert np.array_equal(got[SEQUENTIAL].view(np.uint32), got[WHOLE].view(np.uint32))
    cfg = O.make_config(N=N, lam=lam, G=2, seed=7, T=10, lb=wl.lb, ub=wl.ub)
    take = np.unique(np.concatenate([np.arange(min(N * lam, 20)), np.arange(max(0, N * lam - 20), N * lam)]))
    X = np.stack([O.explosion_row(cfg, before["F"][r // lam, :wl.dim], before["A"][r // lam], r, 1)
                  for r in take])
    want = O.Problem.from_workload(wl).loss_rows(X)
    assert_net_close(wl, X, got[K_SPLIT][take], want, f"{widths} K split")
    assert_net_close(wl, X, got[WHOLE][take], want, f"{widths} whole")
