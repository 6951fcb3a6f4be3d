"""The Newton step's factorisation over the range of FP64: columns scaled by powers of two, so that the
pivots lie between 2^-990 and 2^1012.  Every operation of a step from beta = 0 scales exactly, so it
is the unscaled step divided by the scales, within the bound of the unscaled step (8 p eps cond(A) of
its norm, as both are backward stable)."""
import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p", [2, 17, 70, 201, 330])
@pytest.mark.parametrize("power", [499, 500, -500])
def test_scaled_columns(p, power):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(p)
    n = 6000
    X = np.asfortranarray(rng.standard_normal((n, p)))
    time, event = rng.exponential(1.0, n), (rng.random(n) < 0.7).astype(np.uint8)
    stratum = rng.integers(0, 40, n).astype(np.int32)
    scale = np.ones(p)
    scale[::2] = 2.0 ** power
    print(f"[gpu-test] pivots p={p} power={power}", flush=True)
    out = []
    for x in (X, X * scale):
        with coxmi.CoxModel(np.asfortranarray(x), time, event, stratum, mode=coxmi.COX_NEWTON_REFINE, max_iter=1) as m:
            if not out:
                A = m.evaluate_full(np.zeros(p))[3]
            out.append(np.asarray(m.fit()[0]))
    want, got = out[0], out[1] * scale
    assert np.linalg.norm(got - want) <= 8 * p * np.finfo(np.float64).eps * np.linalg.cond(A) * np.linalg.norm(want)
