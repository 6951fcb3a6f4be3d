"""The scan at the edges of its tiles (1024 threads of 1, 2, 4, 8 or 16 rows, one tile per compute
unit), with arrays that are not 16-byte aligned (no wide accesses), in place, and from more threads at
once than it has sets of synchronisation words.  Inputs are integers, so every sum is exact."""
import threading

import numpy as np
import pytest

from paper_2310_16238_amd import coxmi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _exact(a, f):
    cs = np.r_[0.0, np.cumsum(a)]
    heads = np.r_[True, f[1:] != 0]
    return cs[1:] - cs[:-1][heads][np.cumsum(heads) - 1]


def _inputs(n, heads, seed):
    rng = np.random.default_rng(seed)
    a = rng.integers(-1000, 1000, n).astype(np.float64)
    f = (rng.random(n) < heads).astype(np.uint8) * rng.integers(1, 256, n).astype(np.uint8)
    return a, f


def _scan(a, f, oa=0, of=0, ob=0, in_place=False, stream=None, fn=None):
    n = a.size
    ta = torch.zeros(n + 2, dtype=torch.float64, device="cuda")
    tf = torch.ones(n + 16, dtype=torch.uint8, device="cuda")
    tb = ta if in_place else torch.full((n + 4,), -7.0, dtype=torch.float64, device="cuda")
    ta[oa:oa + n] = torch.tensor(a)
    tf[of:of + n] = torch.tensor(f)
    ob = oa if in_place else ob
    torch.cuda.synchronize()
    (fn or coxmi.cox_segscan_f64)(ta.data_ptr() + 8 * oa, tf.data_ptr() + of, tb.data_ptr() + 8 * ob, n, stream)
    out = tb.cpu().numpy()
    if not in_place:
        assert np.all(out[:ob] == -7.0) and np.all(out[ob + n:] == -7.0)
    return out[ob:ob + n]


@pytest.mark.parametrize("rows", [1, 2, 4, 8, 16])
def test_tile_edges(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tiles = min(torch.cuda.get_device_properties(0).multi_processor_count, 256)
    least = 1 if rows == 1 else tiles * 1024 * rows // 2 + 1
    most = tiles * 1024 * rows
    tile = 1024 * rows
    for n in sorted({least, least + 1, least - least % tile + tile, most - tile + 1, most - 1, most}):
        print(f"[gpu-test] scan rows={rows} n={n}", flush=True)
        for heads in (0.0, 3e-6, 0.05):
            a, f = _inputs(n, heads, n % 1000)
            assert np.array_equal(_scan(a, f), _exact(a, f))


@pytest.mark.parametrize("n", [1, 5, 4097, 300_001, 600_000, 2_500_003])
def test_alignment_and_in_place(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a, f = _inputs(n, 1e-4, n)
    want = _exact(a, f)
    for oa, of, ob in [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 3, 1), (0, 4, 0), (0, 8, 2)]:
        print(f"[gpu-test] scan n={n} offsets {oa} {of} {ob}", flush=True)
        assert np.array_equal(_scan(a, f, oa, of, ob), want)
    assert np.array_equal(_scan(a, f, in_place=True), want)
    assert np.array_equal(_scan(a, f, oa=1, in_place=True), want)
    assert np.array_equal(_scan(a, f, 1, 2, 1, fn=coxmi.cox_segscan_f64_noalloc), want)


def test_more_threads_than_slots():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jobs = [_inputs(n, 1e-5, n) for n in (1000, 70_000, 400_003)]
    want = [_exact(*j) for j in jobs]
    bad = []

    def run(t):
        try:
            s = torch.cuda.Stream()
            for k in range(9):
                i = (t + k) % len(jobs)
                if not np.array_equal(_scan(*jobs[i], stream=s.cuda_stream), want[i]):
                    bad.append((t, k))
        except Exception as e:   # noqa: BLE001 -- reported below
            bad.append(e)

    print("[gpu-test] scans on 40 threads", flush=True)
    ts = [threading.Thread(target=run, args=(t,)) for t in range(40)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
