"""The Newton step's Cholesky factorisation and solves at the edges of its 16-column panels, of its
largest order in LDS (200 columns) and of the 64-column panels beyond, with columns that are not free.

One step from beta0 is compared with numpy's solution of the library's own information matrix and
score.  Both solutions are backward stable, so they differ by at most a few p eps cond(A); the bound
is 8 p eps cond(A) of the step's norm, twice the usual bound of each."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = np.finfo(np.float64).eps


def _data(n, p, seed, dead=()):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, p))
    X[:, list(dead)] = 0.0
    time, event = rng.exponential(1.0, n), (rng.random(n) < 0.7).astype(np.uint8)
    return X, time, event, rng.integers(0, 40, n).astype(np.int32)


@pytest.mark.parametrize("p", [1, 2, 15, 16, 17, 32, 33, 48, 63, 64, 65, 80, 81, 129, 192, 199, 200, 201, 215, 263, 264,
                               265, 328, 329, 513, 640])
def test_one_step(p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dead = [j for j in (0, 5, 16, 40, 64, 150, 199, 200, 230, 512) if 1 < j < p - 1 or (j == 0 and p > 2)]
    X, time, event, stratum = _data(6000, p, p, dead)
    beta0 = np.random.default_rng(p + 1).normal(0.0, 0.2 / np.sqrt(p), p)
    beta0[dead] = 0.0
    print(f"[gpu-test] newton step p={p}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE, max_iter=1) as m:
        _, g, _, info = m.evaluate_full(beta0)
        beta1 = np.asarray(m.fit(beta0)[0])
    free = np.setdiff1d(np.arange(p), dead)
    A = info[np.ix_(free, free)]
    want = np.zeros(p)
    want[free] = -np.linalg.solve(A, g[free])
    got = beta1 - beta0
    bound = 8 * p * EPS * np.linalg.cond(A) * np.linalg.norm(want) + 4 * EPS * np.linalg.norm(beta1)
    assert np.all(got[dead] == 0.0)
    assert np.linalg.norm(got - want) <= bound


@pytest.mark.parametrize("p", [20, 100, 200, 201, 300])
def test_kept_factor(p):
    """A BF16 fit stops refactoring near the end: its last steps are solved from the stored factor.
    It ends where the FP64 fit ends: a score below E 1e-9 (tol 1e-12 on steps of size O(1))."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    X, time, event, stratum = _data(6000, p, p, [3])
    print(f"[gpu-test] kept factor p={p}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE, x_precision=coxmi.COX_BF16,
                        max_iter=50) as m:
        beta = np.asarray(m.fit()[0])
        _, g, _, _ = m.evaluate_full(beta, want_info=False)
    g[3] = 0.0
    assert np.max(np.abs(g)) <= 1e-9 * event.sum()
