"""The Newton step at the largest column counts, where the solve's vector and its staged block need more
than the default 64 KB of LDS (from 4,033 columns): one step solves the library's own information
matrix with a backward error of at most 8 p eps |A|, the bound of the smaller steps, and leaves columns
that are not free at 0."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p", [4032, 4033, 4096])
def test_one_step(p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, dead = 9000, [0, 64, 2047, p - 1]
    rng = np.random.default_rng(p)
    X = np.asfortranarray(rng.standard_normal((p, n)).T)
    X[:, dead] = 0.0
    time, event = rng.exponential(1.0, n), (rng.random(n) < 0.9).astype(np.uint8)
    stratum = rng.integers(0, 9, n).astype(np.int32)
    print(f"[gpu-test] newton step p={p}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE, max_iter=1) as m:
        _, g, _, A = m.evaluate_full(np.zeros(p))
        dx = np.asarray(m.fit()[0])
    free = np.setdiff1d(np.arange(p), dead)
    A, g = A[np.ix_(free, free)], np.asarray(g)[free]
    v = rng.standard_normal(free.size)
    for _ in range(20):
        v = A @ (v / np.linalg.norm(v))
    assert np.all(dx[dead] == 0.0)
    assert np.linalg.norm(A @ dx[free] + g) <= 8 * p * np.finfo(np.float64).eps * np.linalg.norm(v) * np.linalg.norm(dx)
