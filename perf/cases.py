"""Cases that measure the library over the range of work its users give it.

A case is a dict of plain values; ``prepare`` makes what a program holds before the call
(device inputs, a handle), ``run`` is one pass through the public entry points, ``work`` the
bytes and operations such a pass cannot do without and ``exact`` the result in 64 bits from
plain torch, without the library.

Inputs follow the distributions of ``paper_2106_14995_amd.workloads``, drawn on the GPU so
that large batches are made in moments. Kinds of case:

  batch   one batched solve through a handle: the quartic family at one size or at sizes
          log-uniform in [n, nmax], the branch subproblems (n = 6), or the hs45 variant;
          cold starts, with or without the captured graph
  al      the multiplier loop on branch subproblems with line limits (n = 8)
  admm    iterations of the component ADMM from a given state (warm-started branch solves)
  serve   requests given as host arrays to the continuous-batching server, all submitted at
          once, then collected

Mixed sizes are part of the case (drawn from its `mix`); the seed draws the problems.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_14995_amd import tron
from paper_2106_14995_amd import workloads as W

FAMILY = {"qp4": W.QP4, "br6": W.BR6, "hs45m": W.HS45M}
KAPPA, GTOL = 0.1, 1e-6


# ------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------
def batch_case(family, n, batch, nmax=0, graph=False, mix=0, name=None):
    c = {"kind": "batch", "family": family, "n": n, "nmax": nmax or n, "batch": batch, "graph": graph, "mix": mix}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # the smallest calls: a few hundred tiny problems, where latency is everything
        batch_case("qp4", 8, 256, name="qp4_n8_b256"),
        # the branch subproblems of one ADMM iteration on a large grid (bench.py's default)
        batch_case("br6", 6, 65536, name="br6_b65536"),
        # the same for eight load scenarios of that grid solved together: a throughput batch
        batch_case("br6", 6, 524288, name="br6_b524288"),
        # branch subproblems with line limits, each with its own multiplier loop
        {"kind": "al", "batch": 16384, "name": "al_b16384"},
        # uniform batches of the quartic family in the wavefront kernel's range, odd sizes and
        # its two edges among them, up to the largest n (global-memory workspace)
        batch_case("qp4", 24, 10000, name="qp4_n24_b10000"),
        batch_case("qp4", 64, 2048, name="qp4_n64_b2048"),
        batch_case("qp4", 100, 1024, name="qp4_n100_b1024"),
        batch_case("qp4", 200, 512, name="qp4_n200_b512"),
        batch_case("qp4", 512, 512, name="qp4_n512_b512"),
        # mixed sizes in one call, replayed as a graph (bench.py --config uneven)
        batch_case("qp4", 4, 50000, nmax=64, graph=True, mix=3, name="qp4_uneven_b50000"),
        # iterations of the ADMM on a mid-size grid, from a state a little way in
        {"kind": "admm", "nbus": 2000, "nbranch": 3000, "ngen": 500, "iters": 25, "name": "admm_2000bus"},
        # a burst of serving requests of very different sizes, from host memory and back
        {"kind": "serve", "requests": 12, "largest": 1024, "n": 4, "nmax": 128, "mix": 5, "name": "serve_burst"},
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["br6", "qp4", "qp4", "qp4", "mixed", "mixed", "hs45m", "al", "admm", "serve"])
    if kind == "br6":
        return batch_case("br6", 6, _log(rng, 256, 524288), graph=rng.random() < 0.3)
    if kind == "qp4":
        n = _log(rng, 4, 512)
        most = 65536 if n <= 8 else max(256, min(20000, int(6e8 / n ** 3)))
        return batch_case("qp4", n, _log(rng, 64, most), graph=rng.random() < 0.3)
    if kind == "mixed":
        nmax = _log(rng, 24, 400)
        return batch_case("qp4", 4, _log(rng, 100, min(50000, int(1.3e10 / nmax ** 3))), nmax=nmax,
                          graph=rng.random() < 0.5, mix=rng.randint(0, 1 << 20))
    if kind == "hs45m":
        return batch_case("hs45m", _log(rng, 4, 128), _log(rng, 100, 10000), graph=rng.random() < 0.3)
    if kind == "al":
        return {"kind": "al", "batch": _log(rng, 256, 65536)}
    if kind == "admm":
        nbus = _log(rng, 200, 9000)
        return {"kind": "admm", "nbus": nbus, "nbranch": int(nbus * rng.uniform(1.3, 1.8)),
                "ngen": max(1, int(nbus * rng.uniform(0.05, 0.3))), "iters": rng.randint(10, 50)}
    return {"kind": "serve", "requests": rng.randint(4, 16), "largest": _log(rng, 64, 1024), "n": 4,
            "nmax": _log(rng, 32, 128), "mix": rng.randint(0, 1 << 20)}


# ------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(0x5EED + int(seed))
    return g


def _uniform(gen, a, b, *shape):
    return a + (b - a) * torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)


def _sizes(rng, count, nmin, nmax):
    """count sizes, log-uniform in [nmin, nmax]."""
    v = np.exp(rng.uniform(math.log(nmin), math.log(nmax), count))
    return np.clip(np.rint(v), nmin, nmax).astype(np.int32)


def _quartic(gen, count, n):
    """(Q, c, lo, hi) of `count` convex quartic box problems of size n: Q = A'A + 0.1 I."""
    a = torch.randn(count, n, n, generator=gen, device="cuda", dtype=torch.float64)
    q = torch.matmul(a.transpose(1, 2).contiguous(), a)
    q = 0.5 * (q + q.transpose(1, 2)) + 0.1 * torch.eye(n, device="cuda", dtype=torch.float64)
    c = torch.randn(count, n, generator=gen, device="cuda", dtype=torch.float64)
    return q, c, _uniform(gen, -2.0, -0.5, count, n), _uniform(gen, 0.5, 2.0, count, n)


def _quartic_batch(seed, sizes):
    """Packed params, lo, hi, x0 on the device for the given sizes (x0 = 0)."""
    gen = _generator(seed)
    n64 = sizes.astype(np.int64)
    psz = n64 * (n64 + 1) // 2 + n64 + 1
    voff = np.concatenate([[0], np.cumsum(n64)])
    poff = np.concatenate([[0], np.cumsum(psz)])
    params = torch.empty(int(poff[-1]), device="cuda", dtype=torch.float64)
    lo = torch.empty(int(voff[-1]), device="cuda", dtype=torch.float64)
    hi = torch.empty_like(lo)
    for n in np.unique(sizes):
        n = int(n)
        idx = np.nonzero(sizes == n)[0]
        q, c, l, u = _quartic(gen, len(idx), n)
        tri = torch.tril_indices(n, n, device="cuda")
        block = torch.cat([q[:, tri[0], tri[1]], c, torch.full((len(idx), 1), KAPPA, device="cuda", dtype=torch.float64)], 1)
        at = torch.from_numpy(poff[idx]).cuda()[:, None] + torch.arange(block.shape[1], device="cuda")
        params[at] = block
        at = torch.from_numpy(voff[idx]).cuda()[:, None] + torch.arange(n, device="cuda")
        lo[at], hi[at] = l, u
    return params, lo, hi, torch.zeros_like(lo)


def _branches(seed, count, limits=False):
    """Branch subproblems: params, lo, hi, x0 (with `limits`, both ends' line limits as
    equalities with slacks)."""
    gen = _generator(seed)
    u = lambda a, b: _uniform(gen, a, b, count)
    g, b, vi, vj, ti = u(0.5, 5.0), u(-20.0, -1.0), u(0.95, 1.05), u(0.95, 1.05), u(-0.2, 0.2)
    tj = ti + u(-0.25, 0.25)
    flows = _flows(g, b, vi, vj, ti, tj)
    nominal = torch.stack([*flows, vi * vi, vj * vj, ti, tj], 1)
    targets = nominal + 0.05 * torch.randn(count, 8, generator=gen, device="cuda", dtype=torch.float64)
    lam = torch.randn(count, 8, generator=gen, device="cuda", dtype=torch.float64)
    zero, rho = torch.zeros(count, 2, device="cuda", dtype=torch.float64), torch.full((count, 10), 400.0, device="cuda", dtype=torch.float64)
    params = [torch.stack([g, b] * 4, 1), targets, lam, zero, rho]
    lo = [torch.from_numpy(W.BR6_LO).cuda().expand(count, 6)]
    hi = [torch.from_numpy(W.BR6_HI).cuda().expand(count, 6)]
    x0 = [torch.stack([vi, vj, ti, tj, flows[0].clamp(-5, 5), flows[2].clamp(-5, 5)], 1)]
    if limits:
        s2 = torch.stack([flows[0] ** 2 + flows[1] ** 2, flows[2] ** 2 + flows[3] ** 2], 1)
        smax2 = (u(0.85, 1.3) ** 2 * s2.max(1).values)[:, None]
        params += [smax2, zero, torch.full((count, 1), 10.0, device="cuda", dtype=torch.float64)]
        lo.append(zero)
        hi.append(smax2.expand(count, 2))
        x0.append(torch.minimum((smax2 - s2).clamp(min=0.0), smax2))
    return [torch.cat(v, 1).contiguous().view(-1) for v in (params, lo, hi, x0)]


def _flows(g, b, vi, vj, ti, tj):
    """p_ij, q_ij, p_ji, q_ji of a branch with series admittance g + jb and no shunt."""
    wr, wi = vi * vj * torch.cos(ti - tj), vi * vj * torch.sin(ti - tj)
    return (g * (vi * vi - wr) + b * wi, b * (vi * vi - wr) - g * wi,
            g * (vj * vj - wr) - b * wi, b * (vj * vj - wr) + g * wi)


def _hs45(seed, count, n):
    """The hs45 variant with upper bounds U[0.8, 1] i and starts anywhere in the box."""
    gen = _generator(seed)
    hi = torch.arange(1, n + 1, device="cuda", dtype=torch.float64).repeat(count) * _uniform(gen, 0.8, 1.0, count * n)
    x0 = torch.rand(count * n, generator=gen, device="cuda", dtype=torch.float64) * hi
    return torch.zeros(0, device="cuda", dtype=torch.float64), torch.zeros_like(hi), hi, x0


def _batch_inputs(case, seed):
    """(sizes, [params, lo, hi, x0]) of a batch case."""
    count, n = case["batch"], case["n"]
    if case["family"] == "br6":
        return np.full(count, 6, np.int32), _branches(seed, count)
    if case["family"] == "hs45m":
        return np.full(count, n, np.int32), _hs45(seed, count, n)
    sizes = _sizes(np.random.default_rng(case["mix"]), count, n, case["nmax"])
    return sizes, _quartic_batch(seed, sizes)


def _request_sizes(case):
    rng = np.random.default_rng(case["mix"])
    return np.rint(np.exp(rng.uniform(0.0, math.log(case["largest"]), case["requests"]))).astype(int)


def _requests(case, seed):
    """The requests' (n, params, lo, hi, x0) as device tensors (n a host array)."""
    rng = np.random.default_rng([case["mix"], 1])
    out = []
    for k, b in enumerate(_request_sizes(case)):
        sizes = _sizes(rng, int(b), case["n"], case["nmax"])
        out.append((sizes, *_quartic_batch(1000 * seed + k, sizes)))
    return out


# ------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        fam = FAMILY[case["family"]]
        sizes, inputs = _batch_inputs(case, seed)
        opts = tron.options(gtol=GTOL, graph=case["graph"])
        if case["nmax"] > case["n"]:
            h = tron.Batch(fam, sizes, opts=opts)
        else:
            h = tron.Batch(fam, case["n"], batch=case["batch"], opts=opts)
        f64, i32 = torch.float64, torch.int32
        out = dict(x=torch.empty(h.nsum, device="cuda", dtype=f64), f=torch.empty(h.batch, device="cuda", dtype=f64),
                   status=torch.empty(h.batch, device="cuda", dtype=i32), iters=torch.empty(h.batch, device="cuda", dtype=i32))
        return {"kind": kind, "h": h, "inputs": inputs, "out": out}
    if kind == "al":
        return {"kind": kind, "h": tron.Batch(W.BR8L, 8, batch=case["batch"]), "inputs": _branches(seed, case["batch"], limits=True)}
    if kind == "admm":
        a = tron.Admm(W.network(case["nbus"], case["nbranch"], case["ngen"], config_id=1000 + seed))
        a.step(20)
        return {"kind": kind, "h": a, "state": a.get_state(), "iters": case["iters"]}
    reqs = [(r[0], *[t.cpu().numpy() for t in r[1:]]) for r in _requests(case, seed)]
    return {"kind": kind, "h": tron.Server(W.QP4, hbm_budget=256 << 20), "requests": reqs}


def run(state):
    kind, h = state["kind"], state["h"]
    if kind == "batch":
        return h.solve(*state["inputs"], **state["out"])
    if kind == "al":  # the multipliers and the penalty are updated in place: start from the given ones
        params, lo, hi, x0 = state["inputs"]
        params = params.clone()
        return (*h.al_solve(params, lo, hi, x0), params)
    if kind == "admm":
        h.set_state(state["state"])
        resid = h.step(state["iters"])
        return resid, h.get_state()
    tickets = [h.submit(*r) for r in state["requests"]]
    out = []
    for t in tickets:
        h.wait(t)
        r = h.result(t)
        out.append((r["x"], r["f"], r["status"], r["iters"]))
    return out


# ------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------
def _quartic_work(n):
    """(bytes, flops) of one quartic solve of size n: inputs and outputs once; the method's
    operations as counted on these distributions (c factorisations of n^3/3, and products and
    substitutions of about 90 n^2)."""
    c = 3.7 + 0.52 * math.log2(n)
    return 8.0 * (n * (n + 1) // 2 + n + 1 + 4 * n + 1) + 8.0, c * n ** 3 / 3.0 + 90.0 * n * n


def _mean_work(nmin, nmax):
    """The mean of _quartic_work over sizes log-uniform in [nmin, nmax]."""
    pts = [math.exp(math.log(nmin) + (k + 0.5) / 200 * math.log(nmax / nmin)) for k in range(200)]
    w = [_quartic_work(max(nmin, min(nmax, int(round(p))))) for p in pts]
    return sum(b for b, _ in w) / len(w), sum(f for _, f in w) / len(w)


BR6_BYTES, BR6_FLOPS = 496.0, 4786.0  # per branch subproblem: 432 B in, 64 B out


def work(case):
    kind = case["kind"]
    if kind == "batch":
        if case["family"] == "br6":
            b, f = BR6_BYTES, BR6_FLOPS
        elif case["family"] == "hs45m":  # one iteration: an n x n Hessian and a few products with it
            b, f = 8.0 * (4 * case["n"] + 1) + 8.0, 20.0 * case["n"] ** 2
        else:
            b, f = _mean_work(case["n"], case["nmax"]) if case["nmax"] > case["n"] else _quartic_work(case["n"])
        return {"bytes": b * case["batch"], "flops": f * case["batch"]}
    if kind == "al":  # 40 + 3 x 8 doubles in; x, f, viol, three counts and 40 doubles out; about 8 solves each
        return {"bytes": 660.0 * case["batch"], "flops": 8 * 1.6 * BR6_FLOPS * case["batch"]}
    if kind == "admm":  # the state read and written, the network read
        state = 6 * case["ngen"] + 30 * case["nbranch"] + 2 * case["nbus"]
        net = 20 * case["nbranch"] + 6 * case["ngen"] + 4 * case["nbus"]
        return {"bytes": 8.0 * (2 * state + net) * case["iters"], "flops": 0.5 * BR6_FLOPS * case["nbranch"] * case["iters"]}
    b, f = _mean_work(case["n"], case["nmax"])
    count = int(_request_sizes(case).sum())
    return {"bytes": 2.0 * b * count, "flops": f * count}


# ------------------------------------------------------------------------------------
# the result in 64 bits, by another method
# ------------------------------------------------------------------------------------
def _solve_spd(h, b):
    """h^-1 b for a batch of symmetric matrices; a pivot that is not positive counts as its
    magnitude (at least 1e-8), which keeps the step a descent direction."""
    h, n = h.clone(), h.shape[1]
    for j0 in range(0, n, 32):
        j1 = min(j0 + 32, n)
        for j in range(j0, j1):
            if j > j0:
                row = h[:, j, j0:j].contiguous()
                h[:, j:, j] -= torch.matmul(h[:, j:, j0:j], row[:, :, None])[:, :, 0]
            h[:, j:, j] /= h[:, j, j].abs().clamp(min=1e-8).sqrt()[:, None]
        if j1 < n:
            l = h[:, j1:, j0:j1].contiguous()
            h[:, j1:, j1:] -= torch.matmul(l, l.transpose(1, 2).contiguous())
    y = b.clone()
    for j in range(n):
        y[:, j] /= h[:, j, j]
        y[:, j + 1:] -= h[:, j + 1:, j] * y[:, j:j + 1]
    for j in range(n - 1, -1, -1):
        y[:, j] /= h[:, j, j]
        y[:, :j] -= h[:, j, :j] * y[:, j:j + 1]
    return y


def _newton_box(fun, x, lo, hi, iters=60):
    """Projected Newton: minimise fun over the boxes [lo, hi] to rounding, for a batch of
    problems. fun(x, order) gives f (order 0) or f, gradient and Hessian (order 2)."""
    x = torch.minimum(torch.maximum(x, lo), hi)
    eye = torch.eye(x.shape[1], device=x.device, dtype=x.dtype)
    for _ in range(iters):
        f, g, h = fun(x, 2)
        held = ((x <= lo) & (g >= 0)) | ((x >= hi) & (g <= 0))
        for _ in range(3):  # a variable at its bound whose step leads out is held too
            free = (~held).to(x.dtype)
            d = -_solve_spd(h * free[:, :, None] * free[:, None, :] + eye * (1.0 - free)[:, :, None], g * free)
            out = ((x <= lo) & (d < 0)) | ((x >= hi) & (d > 0))
            if not bool((out & ~held).any()):
                break
            held = held | out
        d = d * (~held).to(x.dtype)
        t = torch.ones_like(f)
        for _ in range(40):
            xt = torch.minimum(torch.maximum(x + t[:, None] * d, lo), hi)
            ft = fun(xt, 0)
            ok = ft <= f + 1e-4 * (g * (xt - x)).sum(1) + 1e-13 * f.abs().clamp(min=1.0)
            if bool(ok.all()):
                break
            t = torch.where(ok, t, 0.5 * t)
        xt = torch.where(ok[:, None], xt, x)
        step = float((xt - x).abs().max()) if x.numel() else 0.0
        x = xt
        if step <= 1e-14:
            break
    return x, fun(x, 0)


def _exact_quartic(sizes, inputs):
    """x and f of packed quartic problems, sizes padded to the next power of two (a padding
    variable is fixed at 0)."""
    params, lo, hi, _ = inputs
    n64 = sizes.astype(np.int64)
    voff = np.concatenate([[0], np.cumsum(n64)])
    poff = np.concatenate([[0], np.cumsum(n64 * (n64 + 1) // 2 + n64 + 1)])
    x = torch.empty_like(lo)
    f = torch.empty(len(sizes), device=lo.device, dtype=lo.dtype)
    top = np.array([1 << int(k - 1).bit_length() for k in n64])
    for m in np.unique(top):
        m = int(min(m, sizes.max()))
        which = np.nonzero(top == (1 << (m - 1).bit_length()))[0]
        m = int(sizes[which].max())
        q = torch.zeros(len(which), m, m, device=lo.device, dtype=lo.dtype)
        c, l, u = (torch.zeros(len(which), m, device=lo.device, dtype=lo.dtype) for _ in range(3))
        for n in np.unique(sizes[which]):
            n = int(n)
            k = np.nonzero(sizes[which] == n)[0]
            at = torch.from_numpy(poff[which[k]]).cuda()[:, None] + torch.arange(n * (n + 1) // 2 + n, device="cuda")
            block, tri = params[at], torch.tril_indices(n, n, device="cuda")
            full = torch.zeros(len(k), n, n, device=lo.device, dtype=lo.dtype)
            full[:, tri[0], tri[1]] = block[:, :-n]
            full = full + full.transpose(1, 2) - torch.diag_embed(torch.diagonal(full, dim1=1, dim2=2))
            k = torch.from_numpy(k).cuda()
            q[k, :n, :n], c[k, :n] = full, block[:, -n:]
            at = torch.from_numpy(voff[which][k.cpu().numpy()]).cuda()[:, None] + torch.arange(n, device="cuda")
            l[k, :n], u[k, :n] = lo[at], hi[at]

        def fun(v, order):
            y = torch.matmul(q, v[:, :, None])[:, :, 0]
            val = (v * (0.5 * y + c)).sum(1) + KAPPA * (v ** 4).sum(1)
            if order == 0:
                return val
            return val, y + c + 4.0 * KAPPA * v ** 3, q + torch.diag_embed(12.0 * KAPPA * v * v)

        xs, fs = _newton_box(fun, torch.zeros_like(l), l, u)
        f[torch.from_numpy(which).cuda()] = fs
        for n in np.unique(sizes[which]):
            n = int(n)
            k = np.nonzero(sizes[which] == n)[0]
            at = torch.from_numpy(voff[which[k]]).cuda()[:, None] + torch.arange(n, device="cuda")
            x[at] = xs[torch.from_numpy(k).cuda(), :n]
    return x, f


def _branch_f(x, p):
    """The branch subproblem's objective for one instance (x of 6, p of 36)."""
    flows = _flows(p[0], p[1], x[0], x[1], x[2], x[3])
    y = torch.stack([*flows, x[0] * x[0], x[1] * x[1], x[2], x[3]]) - p[8:16]
    z = torch.stack([x[4] - flows[0], x[5] - flows[2]])
    return (p[16:24] * y + 0.5 * p[26:34] * y * y).sum() + (p[24:26] * z + 0.5 * p[34:36] * z * z).sum()


def _exact_branches(inputs):
    params, lo, hi, x0 = (t.view(-1, k) for t, k in zip(inputs, (36, 6, 6, 6)))
    value, grad, hess = (torch.func.vmap(k) for k in (_branch_f, torch.func.grad(_branch_f), torch.func.hessian(_branch_f)))

    def fun(v, order):
        return value(v, params) if order == 0 else (value(v, params), grad(v, params), hess(v, params))

    x, f = _newton_box(fun, x0, lo, hi, iters=30)
    return x.reshape(-1), f


def exact(case, seed):
    if case["kind"] == "batch":
        sizes, inputs = _batch_inputs(case, seed)
        if case["family"] == "hs45m":  # the upper corner
            hi = inputs[2].view(case["batch"], case["n"])
            f = torch.ones(case["batch"], device="cuda", dtype=torch.float64)
            for k in range(case["n"]):
                f = f * hi[:, k]
            return inputs[2], 120.0 - f, None, None
        x, f = _exact_branches(inputs) if case["family"] == "br6" else _exact_quartic(sizes, inputs)
        return x, f, None, None
    if case["kind"] == "serve":
        out = []
        for r in _requests(case, seed):
            x, f = _exact_quartic(r[0], r[1:])
            out.append((x, f, None, None))
        return out
    # The multiplier loop stops anywhere in its tolerance box (nearly parallel limits leave the
    # multipliers undetermined), and the ADMM's state after a given number of iterations
    # depends on the tolerance of its branch solves: neither has a value of its own.
    return None
