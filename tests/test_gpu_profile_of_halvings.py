"""cox_last_profile of a Newton fit whose steps are halved: the device work of a rejected step counts
too, and after a halving nothing more is queued before the objective is known.  From this start point
the first full step overshoots and is halved several times."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("gamma", [0.0, 1.0])
def test_rejected_steps_count(gamma):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(0)
    n, p = 2000, 3
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time = rng.exponential(1.0, n) * np.exp(-X @ np.array([0.5, -0.3, 0.2]))
    event, stratum = (rng.random(n) < 0.7).astype(np.uint8), rng.integers(0, 20, n).astype(np.int32)
    print(f"[gpu-test] halvings gamma={gamma}", flush=True)
    with coxmi.CoxModel(X, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE, gamma=gamma) as m:
        _, info = m.fit(np.array([4.0, -4.0, 4.0]))
        prof = m.profile()
        _, near = m.fit()
        plain = m.profile()
    rejected = info["coord_evals"] - info["iters"]
    assert info["status"] == coxmi.COX_OK and rejected >= 2
    assert prof["evaluations"] == info["coord_evals"]
    assert prof["solves"] == prof["contractions"]
    assert info["iters"] < prof["solves"] < info["coord_evals"]
    # without halvings nothing is thrown away
    assert near["coord_evals"] == near["iters"] == plain["solves"] == plain["contractions"]
