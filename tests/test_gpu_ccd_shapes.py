"""The persistent kernel's workgroup shapes and its two exchanges against the CPU oracle.

Sizes sit at the edges where the choice of rows per thread, waves per workgroup and one or all
XCDs changes, with strata inside a wave's rows, inside a tile, and across tiles.  Tolerances are
those of the parity tests: g' and g'' within 1e-11 max(1, E) for E events (each sum has E terms
of size O(1)), -log L within 1e-11 max(E, |-log L|).
"""
import numpy as np
import pytest

from oracle import cox_oracle as orc
from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    coxmi.lib()


def _data(n, K, seed):
    rng = np.random.default_rng(seed)
    X = np.asfortranarray(rng.standard_normal((n, 4)))
    X[:, 0] = rng.random(n) < 0.2
    X[:, 3] = 1.0
    time = np.floor(rng.exponential(1.0, n) * 200) / 200
    event = (rng.random(n) < 0.5).astype(np.uint8)
    stratum = (rng.permutation(n).astype(np.int64) * K // n).astype(np.int32)
    return X, time, event, stratum


@pytest.mark.parametrize("n", [1, 255, 513, 2048, 2049, 8191, 16385, 32769, 65537, 131073, 262145, 530000])
@pytest.mark.parametrize("rows", [20, 700, 0])
def test_evaluation_at_every_shape(n, rows):
    K = 1 if rows == 0 else max(1, n // rows)
    X, time, event, stratum = _data(n, K, n + rows)
    # the ones column puts every X beta far below zero: padding rows must not raise the shift
    beta = np.array([0.5, -0.4, 0.3, -40.0])
    L = orc.canonical_layout(time, event, stratum)
    fe = orc.full_eval(orc.to_canonical(X, L), L, beta, want_info=False)
    E = float(event.sum())
    print(f"[gpu-test] ccd shape n={n} K={K}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum) as m:
        obj, g, h = m.evaluate(beta)
        again = m.evaluate(beta)
    assert abs(obj - fe.objective) <= 1e-11 * max(E, abs(fe.objective), 1.0)
    np.testing.assert_allclose(g, fe.grad, atol=1e-11 * max(1.0, E), rtol=0)
    np.testing.assert_allclose(h, fe.hess_diag, atol=1e-11 * max(1.0, E), rtol=0)
    assert again[0] == obj and np.array_equal(again[1], g) and np.array_equal(again[2], h)


@pytest.mark.parametrize("n,K", [(300, 3), (9000, 9), (40000, 2000), (140000, 7)])
def test_indicator_equals_dense(n, K):
    rng = np.random.default_rng(n)
    _, time, event, stratum = _data(n, K, n)
    X = np.asfortranarray((rng.random((n, 6)) < 0.1).astype(np.float64))
    ptr = np.concatenate([[0], np.cumsum((X != 0).sum(0))])
    rows = np.concatenate([np.flatnonzero(X[:, j]) for j in range(6)]).astype(np.int32)
    print(f"[gpu-test] ccd indicator n={n} K={K}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, gamma=0.5) as m:
        dense, _ = m.fit()
    with coxmi.CoxModel.indicator(n, ptr, rows, time, event, stratum, gamma=0.5) as m:
        bits, info = m.fit()
    assert info["status"] == coxmi.COX_OK
    assert np.array_equal(dense, bits)
