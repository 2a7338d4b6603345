"""Performance cases of the evaluation and differentiation paths.

Every case is one pass through the public entry points: an evaluation with
its gradient (``Polynomial.eval_and_diff``), a training step's forward and
reverse pass (``autograd.poly_eval`` and its backward), or many polynomials in
one launch (``Batch.eval_and_diff``).  A case is a dict of plain values:

* ``path``: ``eval``, ``autograd`` or ``batch``;
* ``m``, ``d``: doubles per coefficient and truncation degree;
* ``poly``: ``subsets`` (all r-subsets of n variables) or ``random`` (N
  monomials of nk_lo..nk_hi distinct variables drawn with ``shape_seed``);
* ``cx``: complex series; ``emax``: half of the occurrences get an exponent
  2..emax (1: multilinear);
* batches: ``count`` instances drawn with ``shape_seed`` from the given ranges.

The polynomials' shapes are fixed by the case; the series come from the seed.
"""
import math
from functools import lru_cache

import numpy as np
import torch

from paper_2101_10881_amd import flops as F
from paper_2101_10881_amd import mdpe
from paper_2101_10881_amd import workloads as W
from paper_2101_10881_amd.autograd import poly_eval


def _subsets(n, r, m, d, path="eval", cx=False, emax=1):
    return dict(path=path, poly="subsets", n=n, r=r, m=m, d=d, cx=cx, emax=emax)


def _random(n, N, nk_lo, nk_hi, m, d, shape_seed=1, path="eval", cx=False, emax=1):
    return dict(path=path, poly="random", n=n, N=N, nk_lo=nk_lo, nk_hi=nk_hi, shape_seed=shape_seed, m=m, d=d,
                cx=cx, emax=emax)


def listed():
    return [
        # one small polynomial evaluated again and again (a path tracker's step on a small system): latency counts
        dict(name="rand3_2d_d8", **_random(8, 16, 3, 3, 2, 8)),
        # double double at a low order on a system of medium size: short launches
        dict(name="p1_2d_d31", **_subsets(16, 4, 2, 31)),
        # quad double at an ordinary order
        dict(name="p1_4d_d63", **_subsets(16, 4, 4, 63)),
        # the headline benchmark: 1820 products of 4 of 16 variables, deca double, 153 coefficients
        dict(name="p1_10d_d152", **_subsets(16, 4, 10, 152)),
        # long monomials (64 of 128 variables), quad double: deep chains of dependent products
        dict(name="p2_4d_d64", **_random(128, 128, 64, 64, 4, 64)),
        # the same shape in plain double at the largest order of the published tables
        dict(name="p2_1d_d152", **_random(128, 128, 64, 64, 1, 152)),
        # many short monomials (all 8128 products of 2 of 128 variables), triple double, an odd order
        dict(name="p3_3d_d95", **_subsets(128, 2, 3, 95)),
        # a ragged system: monomials of 1 to 12 variables, odd counts, penta double
        dict(name="ragged_5d_d37", **_random(23, 211, 1, 12, 5, 37, shape_seed=5)),
        # a training step, octo double: forward with the monomial values kept, then the reverse pass
        dict(name="autograd_p1_8d_d32", **_subsets(16, 4, 8, 32, path="autograd")),
        # complex series, double double
        dict(name="complex_p1_2d_d63", **_subsets(16, 4, 2, 63, cx=True)),
        # general exponents (powers and common factors first), quad double
        dict(name="exponents_p1_4d_d31", **_subsets(16, 4, 4, 31, emax=4)),
        # many systems of mixed size, order and precision in one persistent launch
        dict(name="batch_mixed_128", path="batch", count=128, n_lo=8, n_hi=64, N_lo=16, N_hi=1024,
             degrees="8,16,32,64,128", precisions="2,4", shape_seed=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = work(dict(name="", **_subsets(16, 4, 10, 152)))["flops"]
    while True:
        kind = rng.choice(["small", "p1", "p1", "p2", "p3", "ragged", "ragged", "autograd", "complex", "exponents", "batch"])
        m = rng.choice(W.SUPPORTED_M)
        d = _log_int(rng, 5, 191)
        s = rng.randrange(1, 1 << 30)
        if kind == "small":
            c = _random(rng.randint(4, 12), rng.randint(5, 24), 2, 4, rng.choice([1, 2, 3, 4]), _log_int(rng, 3, 16), s)
        elif kind == "p1":
            c = _subsets(rng.randint(9, 17), 4, m, d)
        elif kind == "p2":
            n = rng.randint(40, 128)
            c = _random(n, rng.randint(40, 128), n // 2, n // 2, m, d, s)
        elif kind == "p3":
            c = _subsets(rng.randint(24, 128), 2, m, d)
        elif kind == "ragged":
            lo = rng.randint(1, 3)
            c = _random(rng.randint(13, 40), _log_int(rng, 20, 1500), lo, lo + rng.randint(1, 10), m, d, s)
        elif kind == "autograd":
            c = _subsets(rng.randint(9, 17), rng.randint(2, 4), m, min(d, 96), path="autograd")
        elif kind == "complex":
            c = _subsets(rng.randint(9, 16), rng.randint(2, 4), rng.choice([1, 2, 3, 4, 5]), d, cx=True)
        elif kind == "exponents":
            c = _subsets(rng.randint(9, 16), rng.randint(2, 4), m, d, emax=rng.randint(2, 5))
        else:
            lo, N_lo = rng.randint(8, 30), _log_int(rng, 10, 60)
            ds = sorted({_log_int(rng, 5, 128) for _ in range(rng.randint(2, 5))})
            c = dict(path="batch", count=_log_int(rng, 8, 128), n_lo=lo, n_hi=lo + rng.randint(4, 40), N_lo=N_lo,
                     N_hi=N_lo * rng.randint(2, 16), degrees=",".join(map(str, ds)),
                     precisions=rng.choice(["2,4", "2,4", "1", "2", "3", "4", "8"]), shape_seed=s)
        if work(c)["flops"] <= most:
            return c


# ------------------------------------------------------------------ shapes


@lru_cache(maxsize=64)
def _shape(key):
    """[(n, supports, m, d, exponents or None)] of a case: one entry, or one per batch instance."""
    c = dict(key)
    if c["path"] == "batch":
        rng = np.random.default_rng(c["shape_seed"])
        ds = [int(x) for x in c["degrees"].split(",")]
        ms = [int(x) for x in c["precisions"].split(",")]
        out = []
        for _ in range(c["count"]):
            n = int(rng.integers(c["n_lo"], c["n_hi"] + 1))
            N = int(rng.integers(c["N_lo"], c["N_hi"] + 1))
            d, m = int(rng.choice(ds)), int(rng.choice(ms))
            nk = np.minimum(rng.integers(2, 9, size=N), n)
            out.append((n, W.random_supports(rng, n, N, nk), m, d, None))
        return out
    if c["poly"] == "subsets":
        sup, n = W.all_subsets(c["n"], c["r"]), c["n"]
    else:
        rng, n = np.random.default_rng(c["shape_seed"]), c["n"]
        nk = np.minimum(rng.integers(c["nk_lo"], c["nk_hi"] + 1, size=c["N"]), n)
        sup = W.random_supports(rng, n, c["N"], nk)
    exps = None
    if c["emax"] > 1:
        rng = np.random.default_rng(7)
        q = sum(len(s) for s in sup)
        exps = np.where(rng.uniform(size=q) < 0.5, rng.integers(2, c["emax"] + 1, size=q), 1).astype(np.int32)
    return [(n, sup, c["m"], c["d"], exps)]


def _shapes(case):
    return _shape(tuple(sorted((k, v) for k, v in case.items() if k != "name")))


def _workloads(case, seed):
    """The case's polynomials with their series, as host arrays."""
    out = []
    for q, (n, sup, m, d, exps) in enumerate(_shapes(case)):
        w = W.make("case", m, d, n, sup, seed=(int(seed), q), cx=bool(case.get("cx")))
        w.exps = exps
        out.append(w)
    return out


def _dev(a):
    return torch.from_numpy(a).to("cuda")


# ------------------------------------------------------------- the measured pass


def prepare(case, seed):
    ws = _workloads(case, seed)
    coeff, z = [_dev(w.coeff) for w in ws], [_dev(w.z) for w in ws]
    if case["path"] == "batch":
        # a serving program's state: plans, one batch, one workspace, one flat output buffer
        plans = [mdpe.Plan.for_workload(w, torch.cuda.current_device()) for w in ws]
        batch = mdpe.Batch(plans, tune_cache=mdpe.TUNE_CACHE)
        ws_t = torch.empty(max(batch.info()["workspace_bytes"] // 8, 1), dtype=torch.float64, device="cuda")
        vals = torch.zeros(sum(w.m * (w.d + 1) for w in ws), dtype=torch.float64, device="cuda")
        grads = torch.zeros(sum(w.m * w.n * (w.d + 1) for w in ws), dtype=torch.float64, device="cuda")
        v = list(torch.split(vals, [w.m * (w.d + 1) for w in ws]))
        g = list(torch.split(grads, [w.m * w.n * (w.d + 1) for w in ws]))
        return dict(path="batch", batch=batch, coeff=coeff, z=z, v=v, g=g, ws=ws_t, out={"values": vals, "grads": grads})
    w = ws[0]
    keep = case["path"] == "autograd"
    P = mdpe.Polynomial.for_workload(w, torch.device("cuda", torch.cuda.current_device()), keep_monomials=keep)
    if keep:
        ybar = _dev(W.upstream_adjoint(w.m, w.d, int(seed)))
        return dict(path="autograd", P=P, coeff=coeff[0].requires_grad_(), z=z[0].requires_grad_(), ybar=ybar)
    lead = (2, w.m) if w.cx else (w.m,)
    value = torch.empty(lead + (w.d + 1,), dtype=torch.float64, device="cuda")
    grad = torch.empty(lead + (w.n, w.d + 1), dtype=torch.float64, device="cuda")
    return dict(path="eval", P=P, coeff=coeff[0], z=z[0], value=value, grad=grad)


def run(state):
    if state["path"] == "eval":
        value, grad = state["P"].eval_and_diff(state["coeff"], state["z"], state["value"], state["grad"])
        return {"value": value, "grad": grad}
    if state["path"] == "autograd":
        value, grad = poly_eval(state["coeff"], state["z"], state["P"])
        cbar, zbar = torch.autograd.grad(value, (state["coeff"], state["z"]), state["ybar"])
        return {"value": value.detach(), "grad": grad, "coeff_bar": cbar, "z_bar": zbar}
    state["batch"].eval_and_diff(state["coeff"], state["z"], state["v"], state["g"], state["ws"])
    return state["out"]


# ---------------------------------------------------------------- accounting


def _counts(n, sup, exps):
    """Convolutions, additions and exponent scalings of one polynomial."""
    conv = sum(1 if len(s) == 1 else 3 * len(s) - 3 for s in sup)
    per_var = [0] * n
    for s in sup:
        for v in s:
            per_var[v] += 1
    add = len(sup) + sum(max(0, c - 1) for c in per_var)
    scale = 0
    if exps is not None:
        top, q = [1] * n, 0
        for s in sup:
            for v in s:
                e = int(exps[q])
                q += 1
                top[v] = max(top[v], e - 1)
                conv += e >= 2
                scale += e >= 2
        conv += sum(t - 1 for t in top)
    return conv, add, scale


@lru_cache(maxsize=256)
def _work(key):
    c = dict(key)
    cx, flops, nbytes = bool(c.get("cx")), 0, 0
    for n, sup, m, d, exps in _shape(key):
        conv, add, scale = _counts(n, sup, exps)
        N, per = len(sup), (d + 1) * m * (2 if cx else 1) * 8
        flops += conv * F.conv_flops(m, d, cx) + add * F.add_flops(m, d, cx)
        flops += scale * (d + 1) * (2 if cx else 1) * F.md_flops("mul", m)
        nbytes += per * (N + 1 + n + 1 + n)
        if c["path"] == "autograd":
            # one product of the variables per monomial, then one correlation per input series
            flops += (N + N + n) * F.conv_flops(m, d)
            nbytes += per * (1 + N + 1 + n)
    return {"bytes": float(nbytes), "flops": float(flops)}


def work(case):
    return dict(_work(tuple(sorted((k, v) for k, v in case.items() if k != "name"))))


# ----------------------------------------------------------- plain 64-bit results


def _conv(x, y):
    return np.convolve(x, y)[: x.shape[0]]


def _evaluate(w):
    """value [d+1], gradient [n][d+1] and products of the variables, in float64 (complex128 if complex)."""
    lead = (lambda a: a[0, 0] + 1j * a[1, 0]) if w.cx else (lambda a: a[0])
    a, z = lead(w.coeff), lead(w.z)
    value, grad = a[0].copy(), np.zeros_like(z)
    powers, mono, q = {}, [], 0

    def power(i, p):
        if (i, p) not in powers:
            powers[(i, p)] = z[i] if p == 1 else _conv(power(i, p - 1), z[i])
        return powers[(i, p)]

    for k, s in enumerate(w.supports()):
        es = [1] * len(s) if w.exps is None else [int(e) for e in w.exps[q: q + len(s)]]
        q += len(s)
        ak = a[k + 1]
        for v, e in zip(s, es):
            if e > 1:
                ak = _conv(ak, power(v, e - 1))
        pre = [ak]  # ak * z_1 .. z_j
        for v in s:
            pre.append(_conv(pre[-1], z[v]))
        value = value + pre[-1]
        suf = None  # z_{j+1} .. z_n
        for j in range(len(s) - 1, -1, -1):
            grad[s[j]] += es[j] * (pre[j] if suf is None else _conv(pre[j], suf))
            suf = z[s[j]] if suf is None else _conv(suf, z[s[j]])
        mono.append(suf)
    return value, grad, mono


def _limbs(x, m, cx):
    """A 64-bit array [..., d+1] as the m-double array of the framework: limb 0, the lower limbs zero."""
    if cx:
        return np.stack([_limbs(x.real, m, False), _limbs(x.imag, m, False)])
    out = np.zeros((m,) + x.shape)
    out[0] = x
    return out


def _corr(y, x):
    """sum_j y[s+j] x[j] for every s."""
    return np.convolve(y[::-1], x)[: y.shape[0]][::-1]


def exact(case, seed):
    ws = _workloads(case, seed)
    if case["path"] == "batch":
        if work(case)["flops"] > 3e11:
            return None
        vals, grads = [], []
        for w in ws:
            v, g, _ = _evaluate(w)
            vals.append(_limbs(v, w.m, False).ravel())
            grads.append(_limbs(g, w.m, False).ravel())
        return {"values": np.concatenate(vals), "grads": np.concatenate(grads)}
    w = ws[0]
    v, g, mono = _evaluate(w)
    out = {"value": _limbs(v, w.m, w.cx), "grad": _limbs(g, w.m, w.cx)}
    if case["path"] == "autograd":
        y = W.upstream_adjoint(w.m, w.d, int(seed))[0]
        out["coeff_bar"] = _limbs(np.stack([y] + [_corr(y, x) for x in mono]), w.m, False)
        out["z_bar"] = _limbs(np.stack([_corr(y, x) for x in g]), w.m, False)
    return out
