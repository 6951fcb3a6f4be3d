"""Strata that continue over tiles of rows: the carries of the column pass, with tiles that hold a
head somewhere, at their first row or nowhere, 1 to 200 tiles, column counts around the groups of 4
and 64, and X beta that spans hundreds (the products of the row factors underflow).  Against the
oracle, with the bounds of the full evaluation: score and diagonal within 1e-11 max(1, E) of their
column's scale, the information within 1e-11 of sqrt(a_ii a_jj)."""
import numpy as np
import pytest

from oracle import cox_oracle as orc
from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = {"one": [3000], "two": [1500, 1501], "edges": [513, 511, 1024, 1, 4095, 2, 514, 600], "many": [20_000, 7, 9_000]}


@pytest.mark.parametrize("name", list(SIZES))
@pytest.mark.parametrize("p", [1, 4, 5, 65])
@pytest.mark.parametrize("spread", [0.5, 60.0])
def test_carries(name, p, spread):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(p + 7 * len(name))
    stratum = np.repeat(np.arange(len(SIZES[name]), dtype=np.int32), SIZES[name])
    stratum = stratum[rng.permutation(stratum.size)]
    n = stratum.size
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time = np.floor(rng.exponential(1.0, n) * 500) / 500
    event = (rng.random(n) < 0.6).astype(np.uint8)
    beta = rng.normal(0.0, 1.0, p)
    beta *= spread / np.linalg.norm(beta)
    L = orc.canonical_layout(time, event, stratum)
    fe = orc.full_eval(orc.to_canonical(X, L), L, beta, want_info=True)
    E = float(event.sum())
    print(f"[gpu-test] long strata {name} n={n} p={p} spread={spread}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE) as m:
        obj, g, hd, info = m.evaluate_full(beta)
    big = np.maximum(1.0, np.max(np.abs(X), axis=0))   # every term of the score is at most 2 big, of the diagonal big^2
    assert abs(obj - fe.objective) <= 1e-11 * max(E, abs(fe.objective), 1.0)
    assert np.all(np.abs(g - fe.grad) <= 1e-11 * max(1.0, E) * big)
    assert np.all(np.abs(hd - fe.hess_diag) <= 1e-11 * max(1.0, E) * big ** 2)
    assert np.max(np.abs(info - fe.info) / np.outer(big, big)) <= 1e-11 * max(1.0, E)


@pytest.mark.parametrize("n", [1, 31, 33, 1000, 33_000])
@pytest.mark.parametrize("p", [15, 16, 17, 256, 257])
def test_information_of_row_remainders(n, p):
    """The FP64 products over K ranges whose last chunk of 32 rows is partly or wholly missing:
    one stratum without censoring at beta = 0, against numpy's sums."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n + p)
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time = rng.permutation(n).astype(np.float64)
    with coxmi.CoxModel(X, time, np.ones(n, np.uint8), mode=coxmi.COX_NEWTON_REFINE) as m:
        _, _, _, info = m.evaluate_full(np.zeros(p))
    Xs = X[np.argsort(-time)]
    k = np.arange(1, n + 1)
    lam = np.cumsum((1.0 / k)[::-1])[::-1]
    xbar = np.cumsum(Xs, axis=0) / k[:, None]
    want = (Xs * lam[:, None]).T @ Xs - xbar.T @ xbar
    r = np.sqrt((Xs * Xs * lam[:, None]).sum(0)) + 1.0
    print(f"[gpu-test] information n={n} p={p}", flush=True)
    assert np.max(np.abs(info - want) / np.outer(r, r)) <= 1e-11
