"""The FP64 information on the scale of its own entries: within 1e-11 of sqrt(a_ii a_jj) + sqrt(c_ii c_jj), a and
c its first and second product, the bound of the evaluation's other information tests.  Short strata (a
workgroup each), long ones (tiles and their carries) and X beta that spans hundreds, where a few rows
hold the weight and a sum of squares without weights would be many times the scale."""
import numpy as np
import pytest

from oracle import cox_oracle as orc
from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = {"pairs": [2] * 400, "mixed": [1, 63, 64, 65, 127, 3, 128, 129, 255, 256, 257, 511, 2, 1, 1, 40] * 2,
         "longest": [512, 5, 512, 512], "beyond": [513, 5, 512, 60], "one": [3000], "two": [1500, 1501],
         "edges": [513, 511, 1024, 1, 4095, 2, 514, 600], "many": [20_000, 7, 9_000]}


@pytest.mark.parametrize("name", list(SIZES))
@pytest.mark.parametrize("p", [1, 5, 64, 130, 257])
@pytest.mark.parametrize("spread", [0.5, 60.0])
def test_information(name, p, spread):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(3 * p + len(name))
    stratum = np.repeat(np.arange(len(SIZES[name]), dtype=np.int32), SIZES[name])
    stratum = stratum[rng.permutation(stratum.size)]
    n = stratum.size
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time = np.floor(rng.exponential(1.0, n) * 300) / 300
    event = (rng.random(n) < 0.6).astype(np.uint8)
    beta = rng.normal(0.0, 1.0, p)
    beta *= spread / np.linalg.norm(beta)
    L = orc.canonical_layout(time, event, stratum)
    fe = orc.full_eval(orc.to_canonical(X, L), L, beta, want_info=True)
    print(f"[gpu-test] information {name} n={n} p={p} spread={spread}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE) as m:
        info = m.evaluate_full(beta)[3]
    a, c = (np.sqrt(np.clip(np.diag(v), 0.0, None)) for v in (fe.info_first, fe.info_second))
    assert np.all(np.abs(info - fe.info) <= 1e-11 * (np.outer(a, a) + np.outer(c, c)))
