"""The end of a generation in one launch and in three (needs an MI355X): rows on both
sides of the dispatch line (fireworks x 4-coordinate chunks <= 4096), several populations
finishing in any order, and the target reached by one of them, bit for bit against the
oracle."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_2501_03944_amd import inputs

pytestmark = pytest.mark.gpu


def _objective(X):
    return np.abs(X).max(axis=1).astype(np.float32)


@pytest.mark.parametrize("N,D", [(2, 5), (8, 2048), (8, 2049), (16, 1024), (20, 900)])
@pytest.mark.parametrize("B", [1, 5])
def test_generations_of_an_external_objective(N, D, B):
    """Exact objective values on both sides, so the state has to agree in every bit."""
    torch, M = require_gpu()
    cfg = dict(n_fireworks=N, n_sparks=6, n_guiding=2, n_populations=B, seed=5, max_generations=6)
    g = M.MGFWA((D - 1, 1), (), "mse", external_fitness=True, **cfg)
    X = g.ask()
    start = _objective(X.cpu().numpy()[:, :D])
    g.tell(torch.from_numpy(start).cuda())
    best = start.reshape(B, N).min(axis=1)
    for t in range(1, 4):
        before = {k: np.array(v) for k, v in g.state_numpy().items()}
        for _ in range(2):
            X = g.ask()
            g.tell(torch.from_numpy(_objective(X.cpu().numpy()[:, :D])).cuda())
        s = g.state_numpy()
        Yc, F, Y = s["Yc"], s["F"].reshape(B * N, -1)[:, :D], s["Y"].ravel()
        won = Yc.min(axis=1) < before["Y"].ravel()
        fresh = np.isinf(Y)
        # a firework takes its best candidate where it improves, and is drawn anew where
        # its population has no use for it
        keep = ~fresh
        want = np.where(won, Yc.min(axis=1), before["Y"].ravel())
        assert np.array_equal(Y[keep], want[keep])
        assert np.array_equal(_objective(F)[keep], Y[keep])
        assert np.array_equal(F[keep & ~won], before["F"].reshape(B * N, -1)[keep & ~won, :D])
        assert np.all(np.abs(F) <= 5.0)
        best = np.minimum(best, want.reshape(B, N).min(axis=1))
        assert np.array_equal(s["best_y"].ravel(), best)
        bx = s["best_x"].reshape(B, -1)[:, :D]
        assert np.array_equal(_objective(bx), best)
    g.close()


@pytest.mark.parametrize("B", [1, 7])
def test_target_ends_the_run(B):
    """The first generation whose best value meets the target is the last one."""
    torch, M = require_gpu()
    wl = inputs.teacher_regression()
    free = M.MGFWA.from_workload(wl, n_populations=B, seed=3)
    best = []
    for _ in range(12):
        free.step(1)
        best.append(float(free.state_numpy()["best_y"].min()))
    free.close()
    target = best[5]
    last = 1 + next(i for i, v in enumerate(best) if v <= target)
    g = M.MGFWA.from_workload(wl, n_populations=B, seed=3, target_loss=target)
    g.step(12)
    s = g.state_numpy()
    assert float(s["best_y"].min()) == best[last - 1]
    h = M.MGFWA.from_workload(wl, n_populations=B, seed=3)
    h.step(last)
    t = h.state_numpy()
    for k in ("F", "A", "Y", "best_x", "best_y"):
        assert np.array_equal(s[k], t[k]), k
    g.close()
    h.close()
