"""A row whose X beta is NaN (a NaN in a column with a nonzero coefficient) has no weight in the CCD
path, and the shift of the exponentials is taken over the other rows: with such a row censored, the
other columns' score and curvature are those of the data without it, within the bound of the
evaluation tests (1e-11 E), and a fit from that start point converges with the column pinned."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [300, 5_000, 60_000])
@pytest.mark.parametrize("ties", [coxmi.COX_BRESLOW, coxmi.COX_EFRON])
def test_censored_row(n, ties):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    p, bad = 4, 1
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time, event = rng.exponential(1.0, n), (rng.random(n) < 0.6).astype(np.uint8)
    stratum = rng.integers(0, 5, n).astype(np.int32)
    row = int(np.flatnonzero(event == 0)[7])
    X[row, bad] = np.nan
    beta = np.array([0.2, 0.3, -0.1, 0.05])
    keep = np.arange(n) != row
    others = [0, 2, 3]
    print(f"[gpu-test] NaN row n={n} ties={ties}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, ties=ties, tol=1e-12) as m:
        obj, g, h = m.evaluate(beta)
        fit, info = m.fit(beta)
    with coxmi.CoxModel(np.asfortranarray(X[keep]), time[keep], event[keep], stratum[keep], ties=ties, tol=1e-12) as m:
        obj0, g0, h0 = m.evaluate(beta)
    tol = 1e-11 * event.sum()
    assert abs(obj - obj0) <= 1e-11 * max(event.sum(), abs(obj0))
    assert np.max(np.abs(np.asarray(g)[others] - np.asarray(g0)[others])) <= tol
    assert np.max(np.abs(np.asarray(h)[others] - np.asarray(h0)[others])) <= tol
    # the column with the NaN is pinned at its start value
    assert info["status"] == coxmi.COX_OK and info["n_pinned"] == 1 and fit[bad] == beta[bad]
