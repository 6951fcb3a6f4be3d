"""The proximal model solve at the edges of its 64-coordinate blocks (one block, an odd and an
even number of them, a last block of one): l1 Newton fits against the oracle's CCD optimum.  The
optimum is unique, so the estimates agree to 1e-10 with the same zero pattern, the bound of the
other l1 Newton tests."""
import numpy as np
import pytest

from oracle import cox_oracle as orc
from paper_2310_16238_amd import coxmi, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p", [1, 2, 63, 64, 65, 128, 129, 192, 200])
def test_l1_fit_at_block_edges(p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = synth.make("ar1", 4_000, p, 40, seed=100 + p, beta_sd=0.4)
    pen = np.ones(p, np.uint8)
    if p > 1:
        pen[0] = 0
    L = orc.canonical_layout(d.time, d.event, d.stratum)
    g0 = orc.full_eval(orc.to_canonical(d.X, L), L, np.zeros(p), want_info=False).grad
    gamma = 0.1 * float(np.max(np.abs(g0)))
    print(f"[gpu-test] prox p={p} gamma={gamma:.2f}", flush=True)
    with coxmi.CoxModel(d.X, d.time, d.event, d.stratum, mode=coxmi.COX_NEWTON_REFINE, gamma=gamma, penalize=pen,
                        tol=1e-13, max_iter=300) as m:
        beta, info = m.fit()
        again, _ = m.fit()
    ref = orc.fit_ccd(d.X, d.time, d.event, d.stratum, gamma=gamma, penalize=pen, tol=1e-14, max_sweeps=5000)
    assert ref.converged and info["status"] == coxmi.COX_OK, info
    assert np.array_equal(beta == 0.0, ref.beta == 0.0)
    assert np.max(np.abs(beta - ref.beta)) <= 1e-10 * max(np.max(np.abs(ref.beta)), 1e-300)
    assert np.array_equal(beta, again)
