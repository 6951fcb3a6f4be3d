"""The blocked contraction (P > 256) at the edges of its 256-column blocks and its chunks, BF16 and
FP8, against the oracle's information matrix within the rounding bounds of the narrow cases.  The
two-factor design makes every entry comparable to the diagonal, so a misplaced tile would show."""
import math

import numpy as np
import pytest

from paper_2310_16238_amd import coxmi
from test_gpu_newton import U_BF16, U_FP8, _beta_probe, _check_first_order, _mixed, _oracle_eval, _scale

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", [coxmi.COX_BF16, coxmi.COX_FP8_E4M3], ids=["bf16", "fp8"])
@pytest.mark.parametrize("n,p,K", [(3_001, 257, 3), (2_999, 288, 150), (4_097, 511, 1), (2_500, 512, 125),
                                   (3_333, 513, 7), (60_003, 300, 3000), (2_000, 769, 2)])
def test_information_at_block_edges(n, p, K, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = _mixed(n, p, K, 7)
    beta = _beta_probe(d)
    print(f"[gpu-test] wide contraction n={n} p={p} prec={prec}", flush=True)
    with coxmi.CoxModel(d.X, d.time, d.event, d.stratum, mode=coxmi.COX_NEWTON_REFINE, x_precision=prec) as m:
        obj, g, hd, info = m.evaluate_full(beta)
        again = m.evaluate_full(beta)[3]
    fe = _oracle_eval(d, beta)
    _check_first_order(d, obj, g, hd, fe)
    r = _scale(fe)
    k = math.ceil(d.n / 128) + 16
    lim = (4.5 * U_FP8 if prec == coxmi.COX_FP8_E4M3 else 0.0) + 3.5 * U_BF16 + k * 2.0 ** -24
    worst = float(np.max(np.abs(info - fe.info) / r))
    print(f"[gpu-test]   max |err| / r = {worst:.3e} (bound {lim:.3e})", flush=True)
    assert worst <= lim
    assert np.array_equal(info, info.T) and np.array_equal(info, again)
