"""Timed cases: the calls a user of the library makes, over the sizes they are made at.

A case names a kind of call and its sizes; `prepare` draws the data on the GPU and makes the
handle (or server) such a program keeps, `run` is one call on it.

  scan       the segmented scan primitive on device memory
  evaluate   objective, score and diagonal curvature at a given beta, one scan per column
  ccd        a cyclic-coordinate-descent fit on dense X
  indicator  the same on indicator X (one bit per row)
  full       objective, score and the whole information matrix at a given beta
  newton     a Newton fit (proximal Newton with an l1 weight), information matrix in `precision`
  bootstrap  refits on resampled rows
  serve      a batch of independent fits through the fit server, data in device memory

Designs: "iid" a ones column and N(0,1) columns; "ar1" columns with correlation 0.5^|i-j|;
"binary" 0/1 columns with 5% ones; "heavy" Student-t(3) columns, X beta beyond the range of exp().
Responses: proportional hazards within equal-sized strata, about half of the rows events.
"""
import math

import numpy as np
import torch

from paper_2310_16238_amd import coxmi

_PRECISION = {"f64": coxmi.COX_F64, "bf16": coxmi.COX_BF16, "fp8": coxmi.COX_FP8_E4M3}
_ROOT2 = math.sqrt(2.0)   # the l1 weight of the paper's synthetic fits


def listed():
    return [
        # the scan alone, at the length of the headline data set
        dict(name="scan", kind="scan", n=1_000_003, K=50_000),
        # one look at a small study: launch and synchronisation times count
        dict(name="evaluate_small", kind="evaluate", design="iid", n=10_000, p=10, K=10, ties=True),
        # a small study's l1 fit, follow-up in whole units (ties)
        dict(name="ccd_small", kind="ccd", design="iid", n=10_000, p=10, K=10, ties=True, gamma=_ROOT2),
        # the headline fit: 1e6 rows, 50 columns, strata of 20
        dict(name="ccd_ar1", kind="ccd", design="ar1", n=1_000_000, p=50, K=50_000, ties=False, gamma=0.0),
        # the paper's synthetic grid at its smaller length: 1000 binary covariates, l1
        dict(name="ccd_binary", kind="ccd", design="binary", n=100_000, p=1000, K=5_000, ties=False, gamma=_ROOT2),
        # a propensity-stratified cohort of 97% sparse indicators in 10 long strata
        dict(name="indicator_cohort", kind="indicator", n=946_911, p=300, K=10, gamma=_ROOT2),
        # score and information of a mid-sized model in a few long strata (standard errors at an estimate)
        dict(name="full_f64", kind="full", design="iid", n=200_000, p=100, K=10, ties=False, precision="f64"),
        # Newton with a BF16 information matrix and FP64 refinement, 1e6 x 200
        dict(name="newton_bf16", kind="newton", design="ar1", n=1_000_000, p=200, K=50_000, gamma=0.0, precision="bf16"),
        # the same in FP8 on a wide heavy-tailed design
        dict(name="newton_fp8", kind="newton", design="heavy", n=2_500_000, p=500, K=125_000, gamma=0.0, precision="fp8"),
        # l1 by proximal Newton on 1e6 x 1000 binary covariates
        dict(name="newton_l1", kind="newton", design="binary", n=1_000_000, p=1000, K=50_000, gamma=_ROOT2, precision="bf16"),
        # bootstrap refits of a small model
        dict(name="bootstrap", kind="bootstrap", design="iid", n=20_000, p=20, K=200, reps=8, precision="f64"),
        # a burst of uneven requests: 1e3 to 1e5 rows, 5 to 100 columns
        dict(name="serve", kind="serve", requests=256, lo=1_000, hi=100_000, pmax=100, gamma=0.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "evaluate", "ccd", "ccd", "indicator", "full", "newton", "newton", "bootstrap", "serve"])

    def strata(n):
        return max(1, rng.choice([1, 10, n // 100, n // 20, n // 2]))

    if kind == "scan":
        n = _log(rng, 1_000, 4_000_000)
        return dict(kind=kind, n=n, K=strata(n))
    if kind == "evaluate":
        n = _log(rng, 1_000, 1_000_000)
        return dict(kind=kind, design=rng.choice(["iid", "ar1"]), n=n, p=_log(rng, 5, 100), K=strata(n), ties=rng.random() < 0.5)
    if kind == "ccd":
        if rng.random() < 0.4:
            n = _log(rng, 20_000, 400_000)
            return dict(kind=kind, design="binary", n=n, p=_log(rng, 50, 500), K=strata(n), ties=False, gamma=_ROOT2)
        n = _log(rng, 2_000, 1_000_000)
        return dict(kind=kind, design=rng.choice(["iid", "ar1"]), n=n, p=_log(rng, 5, 50), K=max(1, min(strata(n), n // 20)),
                    ties=rng.random() < 0.5, gamma=rng.choice([0.0, _ROOT2]))
    if kind == "indicator":
        n = _log(rng, 50_000, 946_911)
        return dict(kind=kind, n=n, p=_log(rng, 30, 300), K=strata(n), gamma=_ROOT2)
    if kind == "full":
        n = _log(rng, 5_000, 500_000)
        return dict(kind=kind, design=rng.choice(["iid", "ar1"]), n=n, p=_log(rng, 5, 300), K=strata(n),
                    ties=rng.random() < 0.5, precision="f64")
    if kind == "newton":
        if rng.random() < 0.3:
            n = _log(rng, 100_000, 1_000_000)
            return dict(kind=kind, design="binary", n=n, p=_log(rng, 100, 1000), K=n // 20, gamma=_ROOT2, precision=rng.choice(["bf16", "fp8"]))
        n = _log(rng, 50_000, 1_000_000)
        return dict(kind=kind, design=rng.choice(["iid", "ar1"]), n=n, p=_log(rng, 20, 400), K=max(1, rng.choice([10, n // 100, n // 20])),
                    gamma=0.0, precision=rng.choice(["f64", "bf16", "fp8"]))
    if kind == "bootstrap":
        n = _log(rng, 5_000, 50_000)
        return dict(kind=kind, design="iid", n=n, p=_log(rng, 5, 50), K=n // 100, reps=rng.randint(2, 8), precision=rng.choice(["f64", "bf16"]))
    return dict(kind=kind, requests=_log(rng, 32, 256), lo=1_000, hi=_log(rng, 5_000, 100_000), pmax=_log(rng, 10, 100), gamma=0.0)


# ------------------------------------------------------------------ data

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _exponential(g, n):
    return -torch.log1p(-_rand(g, n))


def _design(g, design, n, p):
    """X as a contiguous (p, n) tensor, and the coefficients the response is drawn with."""
    if design == "iid":
        X = _randn(g, p, n)
        X[0] = 1.0
        return X, 0.5 * _randn(g, p)
    if design == "ar1":
        X = torch.empty(p, n, dtype=torch.float64, device="cuda")
        X[0] = _randn(g, n)
        for j in range(1, p):
            X[j] = 0.5 * X[j - 1] + math.sqrt(0.75) * _randn(g, n)
        return X, 0.5 * _randn(g, p)
    if design == "binary":
        X = torch.empty(p, n, dtype=torch.float64, device="cuda")
        for j in range(0, p, 50):
            X[j:j + 50] = (torch.rand(min(50, p - j), n, generator=g, device="cuda") < 0.05).double()
        return X, _randn(g, p) * (_rand(g, p) < 0.2)
    X = torch.empty(p, n, dtype=torch.float64, device="cuda")   # heavy
    for j in range(p):
        z = torch.randn(4, n, generator=g, device="cuda")
        X[j] = z[0] / z[1:].square().sum(0).sqrt()
    b = torch.zeros(p, dtype=torch.float64, device="cuda")
    b[torch.randperm(p, generator=g, device="cuda")[:max(1, p // 10)]] = _randn(g, max(1, p // 10))
    return X, b


def _response(g, eta, K, ties):
    """(time, event, stratum): log times, or whole hundredths of the times with `ties`."""
    n = eta.numel()
    stratum = (torch.randperm(n, generator=g, device="cuda") * K // n).int()
    lam = (2.0 * _rand(g, K) - 1.0)[stratum.long()] if K > 1 else 0.0
    t = torch.log(_exponential(g, n)) - lam - eta
    c = torch.log(_exponential(g, n)) - lam
    time = torch.minimum(t, c)
    if ties:
        time = torch.floor(torch.exp(time) * 100.0) / 100.0
    return time, (t <= c).to(torch.uint8), stratum


def _data(case, seed):
    g = _gen(seed)
    X, beta = _design(g, case["design"], case["n"], case["p"])
    time, event, stratum = _response(g, beta @ X, case["K"], case.get("ties", False))
    return X, time, event, stratum, beta


def _cohort(case, seed):
    """Indicator columns with 3% ones as compressed columns (host), and the response (host)."""
    g = _gen(seed)
    n, p = case["n"], case["p"]
    b = 0.5 * _randn(g, p) * (_rand(g, p) < 0.2)
    eta = torch.zeros(n, dtype=torch.float64, device="cuda")
    ptr, rows = [0], []
    for j in range(p):
        one = torch.rand(n, generator=g, device="cuda") < 0.03
        eta += b[j] * one
        r = torch.nonzero(one).flatten().int().cpu()
        rows.append(r)
        ptr.append(ptr[-1] + r.numel())
    time, event, stratum = (t.cpu().numpy() for t in _response(g, eta, case["K"], False))
    return np.array(ptr, dtype=np.int64), torch.cat(rows).numpy(), time, event, stratum


def _request_sizes(case):
    """Lengths spread over the logarithm of their range, widths over theirs; the same for every seed."""
    for i in range(case["requests"]):
        a, b = (i * 0.6180339887498949) % 1.0, (i * 0.7548776662466927) % 1.0
        yield int(round(case["lo"] * (case["hi"] / case["lo"]) ** a)), 5 + int(b * (case["pmax"] - 4))


def _requests(case, seed):
    g = _gen(seed)
    for n, p in _request_sizes(case):
        X, beta = _design(g, "iid", n, p)
        yield X, *_response(g, beta @ X, max(1, n // 100), False)


def _counts(case, seed):
    g = np.random.default_rng(seed)
    n = case["n"]
    return g.multinomial(n, np.full(n, 1.0 / n), size=case["reps"]).astype(np.uint32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "scan":
        g = _gen(seed)
        n = case["n"]
        head = torch.zeros(n, dtype=torch.uint8, device="cuda")
        head[torch.randperm(n, generator=g, device="cuda")[:case["K"]]] = 1
        return dict(kind=kind, a=_exponential(g, n), head=head, out=torch.empty(n, dtype=torch.float64, device="cuda"))
    if kind == "serve":
        req = list(_requests(case, seed))
        torch.cuda.synchronize()
        return dict(kind=kind, req=req, server=coxmi.CoxServer(hbm_budget=8 << 30, staging_bytes=256 << 20))
    if kind == "indicator":
        ptr, rows, time, event, stratum = _cohort(case, seed)
        m = coxmi.CoxModel.indicator(case["n"], ptr, rows, time, event, stratum, gamma=case["gamma"])
        return dict(kind=kind, model=m)
    X, time, event, stratum, beta = _data(case, seed)
    newton = kind in ("newton", "bootstrap", "full")
    m = coxmi.CoxModel.from_device(X.T, time, event, stratum, gamma=case.get("gamma", 0.0),
                                   mode=coxmi.COX_NEWTON_REFINE if newton else coxmi.COX_CCD,
                                   x_precision=_PRECISION[case.get("precision", "f64")])
    s = dict(kind=kind, model=m)
    if kind in ("evaluate", "full"):
        s["beta"] = (0.5 * beta).cpu().numpy()
    if kind == "bootstrap":
        s["counts"] = _counts(case, seed)
    return s


def run(s):
    kind = s["kind"]
    if kind == "scan":
        coxmi.cox_segscan_f64(s["a"].data_ptr(), s["head"].data_ptr(), s["out"].data_ptr(), s["a"].numel())
        return s["out"]
    if kind == "serve":
        server = s["server"]
        tickets = [server.submit_device(X.T, time, event, stratum) for X, time, event, stratum in s["req"]]
        got = []
        for t in tickets:
            server.wait(t)
            got.append(server.poll(t))
        return dict(beta=np.concatenate([b for b, _, _ in got]), objective=np.array([i["objective"] for _, i, _ in got]))
    m = s["model"]
    if kind == "evaluate":
        obj, grad, hess = m.evaluate(s["beta"])
        return dict(objective=obj, grad=grad, hess=hess)
    if kind == "full":
        obj, grad, hess, info = m.evaluate_full(s["beta"])
        return dict(objective=obj, grad=grad, hess=hess, info=info)
    if kind == "bootstrap":
        betas, _ = m.bootstrap(s["counts"])
        return betas
    beta, info = m.fit()
    return dict(beta=beta, objective=info["objective"])


def work(case):
    kind = case["kind"]
    if kind == "scan":
        return dict(bytes=17.0 * case["n"], flops=float(case["n"]))
    if kind == "serve":
        sizes = list(_request_sizes(case))
        return dict(bytes=sum(n * (8.0 * p + 13) for n, p in sizes), flops=sum(n * p * (1.5 * (p + 1.0) + 12) for n, p in sizes))
    n, p = case["n"], case["p"]
    if kind == "indicator":
        return dict(bytes=n * (p / 8.0 + 13), flops=12.0 * n * p)
    # X and the keys once; the sums of one evaluation, and of one information matrix (two
    # symmetric products, rows and event groups)
    row = 8.0 * p + 13
    info = 1.5 * p * (p + 1.0)
    if kind in ("evaluate", "ccd"):
        return dict(bytes=n * row, flops=12.0 * n * p)
    if kind == "bootstrap":
        return dict(bytes=n * (row + 4.0 * case["reps"]), flops=n * case["reps"] * (info + 12.0 * p))
    return dict(bytes=n * row + 8.0 * p * p, flops=n * (info + 12.0 * p))


# ------------------------------------------------------------------ values in 64 bits, by plain torch

class _Strata:
    """Rows by stratum and decreasing time, every stratum padded to the longest: (K, m) blocks."""

    def __init__(self, time, event, stratum):
        order = torch.argsort(-time, stable=True)
        order = order[torch.argsort(stratum[order].long(), stable=True)]
        s = stratum[order].long()
        _, s, size = torch.unique_consecutive(s, return_inverse=True, return_counts=True)
        self.K, self.m = size.numel(), int(size.max())
        at = torch.arange(time.numel(), device=time.device) - (torch.cumsum(size, 0) - size)[s]
        self.order, self.slot = order, s * self.m + at
        self.real = self.put(torch.ones_like(time)) > 0
        self.event = self.put(event.double())
        t = self.put(time)
        ends = torch.ones_like(self.real)   # the last row of its tie group
        ends[:, :-1] = (t[:, :-1] != t[:, 1:]) | ~self.real[:, 1:]
        i = torch.where(ends, torch.arange(self.m, device=t.device), self.m)
        self.end = torch.flip(torch.cummin(torch.flip(i, [1]), 1).values, [1]).clamp(max=self.m - 1)

    def put(self, v):
        out = torch.zeros(self.K * self.m, dtype=torch.float64, device=v.device)
        out[self.slot] = v[self.order]
        return out.view(self.K, self.m)

    def terms(self, X, beta, want_info=True):
        """(-log L, score, information or its diagonal) at beta; X is (p, n), sorted into blocks by column chunks."""
        p = X.shape[0]
        eta = self.put(beta @ X)
        masked = torch.where(self.real, eta, -math.inf)
        dev = eta.device
        if self.m <= 128:
            # every event's weights over its own risk set
            rows = torch.arange(self.m, device=dev)
            risk = (rows <= self.end[:, :, None]) & self.real[:, None, :]
            a = torch.where(risk, eta[:, None, :], -math.inf)
            lse = torch.logsumexp(a, 2)
            W = torch.exp(a - lse[:, :, None]) * self.real[:, :, None]
            means = lambda B: torch.bmm(W, B)   # noqa: E731
            weight = torch.bmm(self.event[:, None, :], W)[:, 0]
        else:
            top = masked.max(1, keepdim=True).values
            w = torch.exp(masked - top)
            s0 = torch.cumsum(w, 1).gather(1, self.end)
            lse = torch.log(s0) + top
            hz = torch.zeros_like(w).scatter_add_(1, self.end, self.event / s0)
            weight = w * torch.flip(torch.cumsum(torch.flip(hz, [1]), 1), [1])

            def means(B):
                c = torch.cumsum(w[:, :, None] * B, 1)
                return c.gather(1, self.end[:, :, None].expand_as(B)) / s0[:, :, None]

        obj = (self.event * torch.where(self.event > 0, lse - eta, 0.0)).sum()
        step = max(1, int(2e8) // eta.numel())
        n = X.shape[1]
        xs = torch.empty(p, n, dtype=torch.float64, device=dev) if want_info else None
        zs = torch.empty(p, int((self.event > 0).sum()), dtype=torch.float64, device=dev) if want_info else None
        score, diag = torch.empty(p, dtype=torch.float64, device=dev), torch.empty(p, dtype=torch.float64, device=dev)
        ev, wr = self.event.flatten() > 0, weight.flatten()[self.slot]
        for j in range(0, p, step):
            c = min(step, p - j)
            B = torch.zeros(self.K * self.m, c, dtype=torch.float64, device=dev)
            B[self.slot] = X[j:j + c].T[self.order]
            Z = means(B.view(self.K, self.m, c)).reshape(-1, c)[ev]
            score[j:j + c] = ((weight - self.event).flatten()[:, None] * B).sum(0)
            diag[j:j + c] = (weight.flatten()[:, None] * B * B).sum(0) - (Z * Z).sum(0)
            if want_info:
                xs[j:j + c] = B[self.slot].T
                zs[j:j + c] = Z.T
        if not want_info:
            return obj, score, diag
        return obj, score, (xs * wr) @ xs.T - zs @ zs.T


def _l1_model(H, g, beta, gamma, sweeps=400):
    """The minimiser of g'd + d'Hd/2 + gamma |beta + d|_1, by coordinate descent on the host."""
    H, g, b0 = H.cpu().numpy(), g.cpu().numpy(), beta.cpu().numpy()
    b, r, h = b0.copy(), g.copy(), np.diag(H).copy()
    for _ in range(sweeps):
        most = 0.0
        for j in np.flatnonzero(h > 0):
            u = h[j] * b[j] - r[j]
            new = math.copysign(max(abs(u) - gamma, 0.0), u) / h[j]
            if new != b[j]:
                r += H[j] * (new - b[j])
                most = max(most, abs(new - b[j]))
                b[j] = new
        if most < 1e-15:
            break
    return torch.from_numpy(b - b0).to(beta.device)


def _fit(X, time, event, stratum, gamma):
    """(estimate, penalised objective) by Newton, or proximal Newton, steps; a column without curvature stays at 0."""
    L = _Strata(time, event, stratum)
    beta = torch.zeros(X.shape[0], dtype=torch.float64, device=X.device)
    last, step = math.inf, None
    free = None
    for _ in range(60):
        obj, g, H = L.terms(X, beta)
        obj = float(obj + gamma * beta.abs().sum())
        if step is not None and not obj <= last + 1e-11 * abs(last):
            step = 0.5 * step
            beta = beta - step
            continue
        last = obj
        if free is None:
            free = torch.nonzero(H.diagonal() > 1e-9 * H.diagonal().max()).flatten()
        step = torch.zeros_like(beta)
        Hf, gf = H[free][:, free], g[free]
        step[free] = _l1_model(Hf, gf, beta[free], gamma) if gamma else -torch.linalg.solve(Hf, gf)
        beta = beta + step
        if float(step.abs().max()) <= 1e-12 * max(1.0, float(beta.abs().max())):
            break
    return beta.cpu().numpy(), last


def exact(case, seed):
    kind = case["kind"]
    if kind == "scan":
        s = prepare(case, seed)
        a, head = s["a"], s["head"].bool()
        a, head = a.cpu().numpy(), head.cpu().numpy()
        starts = np.flatnonzero(head)
        if not starts.size or starts[0] != 0:
            starts = np.concatenate([[0], starts])
        ends = np.append(starts[1:], a.size)
        out = np.empty_like(a)
        for i, j in zip(starts, ends):
            np.cumsum(a[i:j], out=out[i:j])
        return torch.from_numpy(out)
    if kind == "serve":
        fits = [_fit(*r, 0.0) for r in _requests(case, seed)]
        return dict(beta=np.concatenate([b for b, _ in fits]), objective=np.array([o for _, o in fits]))
    if kind == "indicator":
        ptr, rows, time, event, stratum = _cohort(case, seed)
        X = torch.zeros(case["p"], case["n"], dtype=torch.float64, device="cuda")
        rows = torch.from_numpy(rows).long().cuda()
        for j in range(case["p"]):
            X[j, rows[ptr[j]:ptr[j + 1]]] = 1.0
        beta, obj = _fit(X, *(torch.from_numpy(v).cuda() for v in (time, event, stratum)), case["gamma"])
        return dict(beta=beta, objective=obj)
    X, time, event, stratum, beta = _data(case, seed)
    if kind in ("evaluate", "full"):
        obj, g, H = _Strata(time, event, stratum).terms(X, 0.5 * beta, kind == "full")
        out = dict(objective=float(obj), grad=g.cpu().numpy(), hess=(H.diagonal() if kind == "full" else H).cpu().numpy())
        return dict(out, info=H.cpu().numpy()) if kind == "full" else out
    if kind == "bootstrap":
        betas = []
        for c in _counts(case, seed):
            i = torch.repeat_interleave(torch.arange(case["n"], device="cuda"), torch.from_numpy(c.astype(np.int64)).cuda())
            betas.append(_fit(X[:, i].contiguous(), time[i], event[i], stratum[i], 0.0)[0])
        return np.stack(betas)
    beta, obj = _fit(X, time, event, stratum, case["gamma"])
    return dict(beta=beta, objective=obj)
