"""The one-launch evaluation of whole strata per workgroup: column counts at the edges of its
64-column groups, strata up to its longest (512 rows) and one beyond (the tiled kernels), against
the oracle.  Bounds as for the full evaluation: score and diagonal within 1e-11 max(1, E), -log L
within 1e-11 max(E, |-log L|) (E events, each sum has E terms of size O(1)); the FP64 information
within 1e-11 of sqrt(a_ii a_jj), a the diagonal of its first product."""
import numpy as np
import pytest

from oracle import cox_oracle as orc
from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _strata(rng, sizes):
    s = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    return s[rng.permutation(s.size)]


SIZES = {"pairs": [2] * 400, "mixed": [1, 63, 64, 65, 127, 3, 128, 129, 255, 256, 257, 511, 2, 1, 1, 40] * 2,
         "longest": [512, 5, 512, 512], "beyond": [513, 5, 512, 60], "one": [1], "single": [300]}


@pytest.mark.parametrize("name", list(SIZES))
@pytest.mark.parametrize("p", [1, 7, 63, 64, 65, 130, 257, 513])
def test_evaluation(name, p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(p + len(name))
    stratum = _strata(rng, SIZES[name])
    n = stratum.size
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time = np.floor(rng.exponential(1.0, n) * 60) / 60
    event = (rng.random(n) < 0.6).astype(np.uint8)
    beta = rng.normal(0.0, 0.4 / np.sqrt(p), p)
    beta[rng.random(p) < 0.3] = 0.0
    L = orc.canonical_layout(time, event, stratum)
    fe = orc.full_eval(orc.to_canonical(X, L), L, beta, want_info=True)
    E = float(event.sum())
    print(f"[gpu-test] segments {name} n={n} p={p}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE) as m:
        obj, g, hd, info = m.evaluate_full(beta)
        obj2, g2, _, _ = m.evaluate_full(beta, want_info=False)
        haz = m.baseline_hazard(beta)
        obj0, g0, _, _ = m.evaluate_full(np.zeros(p))
    tol = 1e-11 * max(1.0, E)
    assert abs(obj - fe.objective) <= 1e-11 * max(E, abs(fe.objective), 1.0) and obj2 == obj
    np.testing.assert_allclose(g, fe.grad, atol=tol, rtol=0)
    np.testing.assert_allclose(g2, fe.grad, atol=tol, rtol=0)
    np.testing.assert_allclose(hd, fe.hess_diag, atol=tol, rtol=0)
    r = np.sqrt(np.outer((X * X).sum(0), (X * X).sum(0))) + 1.0
    assert np.max(np.abs(info - fe.info) / r) <= 1e-11
    z = orc.full_eval(orc.to_canonical(X, L), L, np.zeros(p), want_info=False)
    np.testing.assert_allclose(g0, z.grad, atol=tol, rtol=0)
    # martingale residuals sum to zero in every stratum
    resid = event - np.exp(X @ beta) * haz
    assert np.max(np.abs(np.bincount(stratum, resid))) <= tol
