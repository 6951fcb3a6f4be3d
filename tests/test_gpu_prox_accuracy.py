"""The estimates of an l1 Newton fit are the model's minimum to the last few units of FP64.

At a fit's end the model there (the library's own score and information) is minimised once more, in
extended precision on the host: what is left to move is the fit's rounding.  With u = eps / 2, a
coordinate's solution takes five roundings at the size of a |beta| (a beta - g, the weight, the sum of
the other moves, the inverse, the product), within 8 u |beta| together.  Its score is a sum of E terms
of size sd(x), each within 32 u of it (X beta of size 10, its exponential, the risk-set sums), together
within 32 u sqrt(E) sd(x), over the curvature E var(x): 32 u / sqrt(E).  The inverse of H with rows
divided by its diagonal carries these to the others; they are independent, so they add in squares:
bound six times the root."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p", [64, 150, 300])
def test_fit_is_the_models_minimum(p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gamma = 1.0
    d = synth.make("ar1", 8_000, p, 80, seed=p, beta_sd=0.3)
    print(f"[gpu-test] l1 accuracy p={p}", flush=True)
    with coxmi.CoxModel(d.X, d.time, d.event, d.stratum, mode=coxmi.COX_NEWTON_REFINE, gamma=gamma, tol=1e-14,
                        max_iter=40) as m:
        beta = np.asarray(m.fit()[0])
        _, g, _, H = m.evaluate_full(beta)
    Hl, gl, b = H.astype(np.longdouble), g.astype(np.longdouble), beta.astype(np.longdouble)
    D, HD = np.zeros(p, np.longdouble), np.zeros(p, np.longdouble)
    for _ in range(400):
        most = 0.0
        for j in range(p):
            a = Hl[j, j]
            u = a * (b[j] + D[j]) - gl[j] - HD[j]
            z = np.sign(u) * max(abs(u) - gamma, 0.0) / a
            move = z - b[j] - D[j]
            if move != 0.0:
                D[j] += move
                HD += Hl[j] * move
                most = max(most, abs(move))
        if most < 1e-18:
            break
    u = np.finfo(np.float64).eps / 2
    carry = np.linalg.inv(H / np.diag(H)[:, None])
    own = 8 * u * (np.abs(beta) + 4 / np.sqrt(d.event.sum()))
    bound = 6 * np.max(np.sqrt((carry ** 2) @ own ** 2))
    print(f"  left {float(np.max(np.abs(D))):.2e} bound {bound:.2e}", flush=True)
    assert np.count_nonzero(beta) > p // 2
    assert float(np.max(np.abs(D))) <= bound
