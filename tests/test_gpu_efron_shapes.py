"""Efron's ties in the persistent kernel over its workgroup shapes (their own three among them: 512 threads of
1, 2 and 4 rows), with strata inside a wave's rows, inside a tile and over tiles, on dense, indicator and
sparse X: objective, score and curvature against the tiled full evaluation, within the bound of the
evaluation tests (1e-11 E on 0/1 columns), the three kinds of X the same to the last bits.

Large groups of ties are taken where a wave has few rows: a coordinate with groups of 50 events takes at most
4.5 times one without ties (2.6 with 512 threads of one row, 7.4 with eight rows per thread)."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _data(n, K, per_unit, seed):
    rng = np.random.default_rng(seed)
    X = np.asfortranarray((rng.random((n, 3)) < 0.3).astype(np.float64))
    time = np.floor(rng.exponential(1.0, n) * per_unit)
    return X, time, (rng.random(n) < 0.5).astype(np.uint8), rng.integers(0, K, n).astype(np.int32)


@pytest.mark.parametrize("n", [700, 5_000, 40_000, 120_000, 200_000, 400_000, 600_000, 1_200_000])
@pytest.mark.parametrize("rows", [20, 400, 10_000, 10**9])
@pytest.mark.parametrize("per_unit", [5, 1000])
def test_evaluation(n, rows, per_unit):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    X, time, event, stratum = _data(n, max(1, n // rows), per_unit, n)
    beta = np.array([0.3, -0.2, 0.1])
    S = sp.csc_matrix(X)
    col, row = S.indptr.astype(np.int64), S.indices.astype(np.int32)
    print(f"[gpu-test] Efron shapes n={n} rows={rows} per_unit={per_unit}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, ties=coxmi.COX_EFRON) as m:
        got = m.evaluate(beta)
        want = m.evaluate_full(beta, want_info=False)
    with coxmi.CoxModel(X, time, event, stratum, ties=coxmi.COX_EFRON, mode=coxmi.COX_NEWTON_REFINE) as m:
        newton = m.evaluate(beta)
    with coxmi.CoxModel.indicator(n, col, row, time, event, stratum, ties=coxmi.COX_EFRON) as m:
        ind = m.evaluate(beta)
    with coxmi.CoxModel.sparse(n, col, row, S.data, time, event, stratum, ties=coxmi.COX_EFRON) as m:
        sparse = m.evaluate(beta)
    E = float(event.sum())
    for other in (got, newton, ind, sparse):
        assert abs(other[0] - want[0]) <= 1e-11 * max(E, abs(want[0]))
        for a, b in zip(other[1:], want[1:]):
            assert np.max(np.abs(np.asarray(a) - np.asarray(b))) <= 1e-11 * E
    for a, b in zip(got, sparse):
        assert np.array_equal(a, b)


def test_large_groups_have_few_rows_per_wave():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    X, time, event, _ = _data(100_000, 1, 1000, 1)
    ms = []
    for ties in (coxmi.COX_BRESLOW, coxmi.COX_EFRON):
        with coxmi.CoxModel(X, time, event, None, ties=ties) as m:
            best = np.inf
            for _ in range(20):
                m.evaluate(np.zeros(3))
                best = min(best, m.kernel_ms())
        ms.append(best)
    print(f"[gpu-test] Breslow {1e3 * ms[0]:.1f} us, Efron {1e3 * ms[1]:.1f} us", flush=True)
    assert ms[1] <= 4.5 * ms[0]
