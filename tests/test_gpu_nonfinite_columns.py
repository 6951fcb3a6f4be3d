"""Columns whose information is not finite (one NaN, one infinity) or zero stay at 0 and touch no
other column: every kind of fit equals the fit without those columns.  They sit inside, at the edges of
and alone in the 64-coordinate blocks of the proximal solve, the panels of the Cholesky factorisation
and the 32- and 256-column tiles of the products, in short strata (evaluated whole by one workgroup)
and long ones (tiles).  Both fits stop at steps below 1e-13 on an FP64 score, so the estimates agree to
1e-10 with the same zero pattern, the bound of the other Newton tests."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BAD = {5: (2,), 10: (0, 4), 65: (64,), 130: (0, 63, 64, 70, 129), 300: (7, 255, 256, 299)}
PREC = {"f64": coxmi.COX_F64, "bf16": coxmi.COX_BF16, "fp8": coxmi.COX_FP8_E4M3}


def _data(p, long_strata, seed):
    rng = np.random.default_rng(seed)
    n = 6000
    X = np.asfortranarray(rng.standard_normal((n, p)))
    good = np.setdiff1d(np.arange(p), BAD[p])
    eta = X[:, good] @ (rng.normal(0.0, 0.4, good.size) * (rng.random(good.size) < 0.3))
    t, c = rng.exponential(1.0, n) * np.exp(-eta), rng.exponential(1.0, n)
    stratum = (np.arange(n) % (3 if long_strata else 300)).astype(np.int32)
    return X, np.minimum(t, c), (t <= c).astype(np.uint8), stratum, good


def _fit(X, time, event, stratum, gamma, mode, precision):
    with coxmi.CoxModel(np.asfortranarray(X), time, event, stratum, mode=mode, gamma=gamma, x_precision=precision,
                        tol=1e-13, max_iter=2000 if mode == coxmi.COX_CCD else 300) as m:
        beta, info = m.fit()
    return np.asarray(beta), info


@pytest.mark.parametrize("p", list(BAD))
@pytest.mark.parametrize("what", ["nan", "inf", "zero"])
@pytest.mark.parametrize("penalised", [True, False])
@pytest.mark.parametrize("precision", [*PREC, "ccd"])
def test_other_columns_are_not_touched(p, what, penalised, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if precision == "ccd" and p > 65:
        pytest.skip("thousands of sweeps")
    mode = coxmi.COX_CCD if precision == "ccd" else coxmi.COX_NEWTON_REFINE
    for long_strata in (False, True):
        X, time, event, stratum, good = _data(p, long_strata, p)
        print(f"[gpu-test] {what} columns p={p} l1={penalised} {precision} long={long_strata}", flush=True)
        with coxmi.CoxModel(np.asfortranarray(X[:, good]), time, event, stratum, mode=coxmi.COX_NEWTON_REFINE) as m:
            g0 = m.evaluate_full(np.zeros(good.size), want_info=False)[1]
        gamma = 0.1 * float(np.max(np.abs(g0))) if penalised else 0.0
        want, winfo = _fit(X[:, good], time, event, stratum, gamma, mode, PREC.get(precision, coxmi.COX_F64))
        for k, j in enumerate(BAD[p]):
            X[(37 * k + 5) % X.shape[0], j] = {"nan": np.nan, "inf": np.inf, "zero": 0.0}[what]
            if what == "zero":
                X[:, j] = 0.0
        got, info = _fit(X, time, event, stratum, gamma, mode, PREC.get(precision, coxmi.COX_F64))
        assert winfo["status"] == coxmi.COX_OK and info["status"] == coxmi.COX_OK
        assert info["n_pinned"] == len(BAD[p])
        assert np.all(got[list(BAD[p])] == 0.0)
        assert np.count_nonzero(want) > 0 and np.array_equal(got[good] == 0.0, want == 0.0)
        assert np.max(np.abs(got[good] - want)) <= 1e-10 * np.max(np.abs(want))
