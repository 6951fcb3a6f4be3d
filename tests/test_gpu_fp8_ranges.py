"""The FP8 contraction around its one-pass kernel's last column count (320) and with few rows for many columns,
where the blocks' K ranges are fewer and longer: within the rounding bound of the other FP8 information
tests, twice the same bits.  And the reason: 20,000 rows of 800 columns cost less than the same in BF16
(0.62 times; 0.98 with a partial written and read for every 128 rows; bound 0.85)."""
import math

import numpy as np
import pytest

from paper_2310_16238_amd import coxmi
from test_gpu_newton import U_BF16, U_FP8, _beta_probe, _check_first_order, _mixed, _oracle_eval, _scale

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,p,K", [(300, 320, 3), (300, 321, 3), (9_999, 319, 1), (9_999, 320, 500), (9_999, 321, 500),
                                   (5_001, 352, 2), (20_011, 800, 1000), (1_025, 1000, 5)])
def test_information(n, p, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = _mixed(n, p, K, 11)
    beta = _beta_probe(d)
    print(f"[gpu-test] FP8 ranges n={n} p={p}", flush=True)
    with coxmi.CoxModel(d.X, d.time, d.event, d.stratum, mode=coxmi.COX_NEWTON_REFINE,
                        x_precision=coxmi.COX_FP8_E4M3) as m:
        obj, g, hd, info = m.evaluate_full(beta)
        again = m.evaluate_full(beta)[3]
    fe = _oracle_eval(d, beta)
    _check_first_order(d, obj, g, hd, fe)
    lim = 4.5 * U_FP8 + 3.5 * U_BF16 + (math.ceil(d.n / 128) + 16) * 2.0 ** -24
    assert np.all(np.abs(info - fe.info) <= lim * _scale(fe))
    assert np.array_equal(info, info.T) and np.array_equal(info, again)


def test_few_rows_of_many_columns():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, p = 20_000, 800
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(p, n, generator=g, device="cuda", dtype=torch.float64)
    time = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    event = (torch.rand(n, generator=g, device="cuda") < 0.5).to(torch.uint8)
    stratum = (torch.arange(n, device="cuda") // 20).int()
    ms = []
    for precision in (coxmi.COX_BF16, coxmi.COX_FP8_E4M3):
        with coxmi.CoxModel.from_device(X.T, time, event, stratum, mode=coxmi.COX_NEWTON_REFINE,
                                        x_precision=precision) as m:
            best = np.inf
            for _ in range(10):
                m.evaluate_full(np.zeros(p))
                best = min(best, m.profile()["contraction_ms"])
        ms.append(best)
    print(f"[gpu-test] 20,000 x 800: BF16 {1e3 * ms[0]:.0f} us, FP8 {1e3 * ms[1]:.0f} us", flush=True)
    assert ms[1] <= 0.85 * ms[0]
