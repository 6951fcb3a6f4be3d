"""Where an evaluation goes by segments of whole strata, where by tiles, and where by one with xbar and by the
other without (2,100 rows in strata of 350): objective, score and information against the oracle with the
bounds of the evaluation tests, fits in every precision to a score below E 1e-9, residuals that sum to
zero.  And the reason for the rule: strata that leave most of a segment's waves idle cost no more than
longer ones that go by tiles (0.9 times; by segments 1.7 times; bound 1.3)."""
import numpy as np
import pytest

from oracle import cox_oracle as orc
from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PREC = {"f64": coxmi.COX_F64, "bf16": coxmi.COX_BF16, "fp8": coxmi.COX_FP8_E4M3}


@pytest.mark.parametrize("rows", [20, 90, 180, 250, 350, 500])
@pytest.mark.parametrize("p", [5, 20, 70])
@pytest.mark.parametrize("precision", list(PREC))
def test_either_way(rows, p, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 2100
    rng = np.random.default_rng(rows + p)
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time, event = rng.exponential(1.0, n), (rng.random(n) < 0.6).astype(np.uint8)
    stratum = (np.arange(n) // rows).astype(np.int32)
    beta = rng.normal(0.0, 0.3 / np.sqrt(p), p)
    L = orc.canonical_layout(time, event, stratum)
    fe = orc.full_eval(orc.to_canonical(X, L), L, beta, want_info=True)
    E = float(event.sum())
    print(f"[gpu-test] segment rule rows={rows} p={p} {precision}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE, x_precision=PREC[precision],
                        max_iter=60) as m:
        obj, g, hd, info = m.evaluate_full(beta)
        haz = m.baseline_hazard(beta)
        fit, fi = m.fit()
        g1 = m.evaluate_full(fit, want_info=False)[1]
    assert abs(obj - fe.objective) <= 1e-11 * max(E, abs(fe.objective))
    assert np.max(np.abs(g - fe.grad)) <= 1e-11 * E * np.max(np.abs(X))
    assert np.max(np.abs(hd - fe.hess_diag)) <= 1e-11 * E * np.max(np.abs(X)) ** 2
    a, c = (np.sqrt(np.clip(np.diag(v), 0.0, None)) for v in (fe.info_first, fe.info_second))
    # as in the information tests: 1e-11, 3.5 and 4.5 + 3.5 unit roundoffs of the stored operands
    bound = {"f64": 1e-11, "bf16": 3.5 * 2.0 ** -8, "fp8": 4.5 * 2.0 ** -3 + 3.5 * 2.0 ** -8}[precision]
    assert np.all(np.abs(info - fe.info) <= bound * (np.outer(a, a) + np.outer(c, c)))
    assert fi["status"] == coxmi.COX_OK and np.max(np.abs(g1)) <= 1e-9 * E
    assert np.max(np.abs(np.bincount(stratum, event - np.exp(X @ beta) * haz))) <= 1e-11 * E


def test_half_empty_segments():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, p = 500_000, 20
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(p, n, generator=g, device="cuda", dtype=torch.float64)
    time = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    event = (torch.rand(n, generator=g, device="cuda") < 0.5).to(torch.uint8)
    ms = {}
    for rows in (400, 600):
        stratum = (torch.arange(n, device="cuda") // rows).int()
        with coxmi.CoxModel.from_device(X.T, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE) as m:
            ms[rows] = np.inf
            for _ in range(10):
                m.evaluate_full(np.zeros(p), want_info=False)
                ms[rows] = min(ms[rows], m.profile()["evaluation_ms"])
    print(f"[gpu-test] strata of 400 rows {1e3 * ms[400]:.0f} us, of 600 rows {1e3 * ms[600]:.0f} us", flush=True)
    assert ms[400] <= 1.3 * ms[600]
