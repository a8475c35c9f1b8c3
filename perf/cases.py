"""Timed workloads of the framework, through its public entry points.

`listed()` names the workloads, `draw()` gives more of the same ranges,
`prepare()` makes what a program holds before the call (matrices, right-hand
sides, point buffers, a context), `run()` is one pass, `work()` the bytes and
operations a pass cannot do without, and `exact()` the same outputs in plain
64-bit torch.

Kinds of case:
  solve    lupp_batched_solve on one uniform batch of n x n systems
           (n = 2..32, 1000 to 2^20 systems, AoS or interleaved). Matrices are
           N(0, 1), right-hand sides b = A x with x ~ U(-1, 1). The solve
           overwrites b; where the factors are asked for it overwrites A too.
           A program that solves again with the same data restores what the
           call overwrites, and so does a pass: b always, A with the factors.
  ragged   lupp_batched_solve_ragged, sizes 2..32 mixed in one batch, each equally often.
  grouped  lupp_batched_solve_grouped, a burst of uniform batches of different
           sizes (the serving loop's merged solves).
  newton   constitutive_update, the fused Newton update of integration points
           from a committed state (restored before the pass, as a global
           iteration restarts from the last committed step).
"""
from __future__ import annotations

import math

import torch

import paper_2609_15217_amd.lupp as lupp

MI = 1 << 20
# rows of one matrix element of an interleaved batch: padded off a power of two
SOA_PAD = 192
SOLVES_PER_POINT = 17.7  # mean Newton solves of a point at increments of 2e-3


def listed():
    return [
        # one small call, as a host program issues them: launch and latency
        {"name": "solve_aos_n8_4096", "kind": "solve", "n": 8, "batch": 4096, "layout": "aos",
         "fma": False, "factors": False, "pad": 0},
        # a small ragged-edged call of larger systems: the length of one solve's chain
        {"name": "solve_soa_n21_5003", "kind": "solve", "n": 21, "batch": 5003, "layout": "soa",
         "fma": False, "factors": False, "pad": 0},
        # tiny systems in a user's natural (packed) layout
        {"name": "solve_aos_n5_1m", "kind": "solve", "n": 5, "batch": MI, "layout": "aos",
         "fma": False, "factors": False, "pad": 0},
        # the size of the constitutive laws' systems, factors kept (getrf role)
        {"name": "solve_aos_n12_1m_factors", "kind": "solve", "n": 12, "batch": MI,
         "layout": "aos", "fma": False, "factors": True, "pad": 0},
        # interleaved batch of a middle size
        {"name": "solve_soa_n16_1m", "kind": "solve", "n": 16, "batch": MI, "layout": "soa",
         "fma": False, "factors": False, "pad": SOA_PAD},
        # an odd size and an odd count in fused multiply-add arithmetic
        {"name": "solve_aos_n17_300007_fma", "kind": "solve", "n": 17, "batch": 300007,
         "layout": "aos", "fma": True, "factors": False, "pad": 0},
        # interleaved batch of large systems, factors kept
        {"name": "solve_soa_n24_1m_factors", "kind": "solve", "n": 24, "batch": MI,
         "layout": "soa", "fma": False, "factors": True, "pad": SOA_PAD},
        # the largest size, packed
        {"name": "solve_aos_n32_1m", "kind": "solve", "n": 32, "batch": MI, "layout": "aos",
         "fma": False, "factors": False, "pad": 0},
        # mixed sizes in one call
        {"name": "ragged_2m", "kind": "ragged", "batch": 2_000_000},
        # a burst of waiting solve requests served together
        {"name": "grouped_24", "kind": "grouped", "groups": 24, "burst": 24, "lo": 1000,
         "hi": 30000},
        # fused Newton updates: 7 unknowns, a large mesh
        {"name": "newton7_1m", "kind": "newton", "law": 7, "points": MI, "amp": 2e-3,
         "tangent": False},
        # 13 unknowns with the consistent tangent, a middle-sized mesh
        {"name": "newton13_tangent_200k", "kind": "newton", "law": 13, "points": 200_003,
         "amp": 2e-3, "tangent": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.55:
        n = rng.randint(2, 32)
        factors = rng.random() < 0.35
        hi = min(MI, MI * 24 * 24 // (n * n)) if factors else MI
        layout = rng.choice(["aos", "soa"])
        return {"kind": "solve", "n": n, "batch": _log_int(rng, 1000, hi), "layout": layout,
                "fma": rng.random() < 0.25, "factors": factors,
                "pad": rng.choice([0, SOA_PAD]) if layout == "soa" else 0}
    if u < 0.67:
        return {"kind": "ragged", "batch": _log_int(rng, 20_000, 2_000_000)}
    if u < 0.80:
        return {"kind": "grouped", "groups": rng.randint(4, 32), "burst": rng.randint(1, 10 ** 6),
                "lo": 1000, "hi": 30000}
    law = rng.choice([7, 13])
    return {"kind": "newton", "law": law, "points": _log_int(rng, 1000, MI if law == 7 else MI // 4),
            "amp": rng.choice([2e-3, 2e-4]), "tangent": rng.random() < 0.4}


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _systems(n, batch, g):
    """A (batch, n, n) read [s][j][i] and b = A x (batch, n)."""
    A = torch.randn((batch, n, n), generator=g, dtype=torch.float64, device="cuda")
    x = torch.rand((batch, n), generator=g, dtype=torch.float64, device="cuda") * 2 - 1
    b = torch.zeros((batch, n), dtype=torch.float64, device="cuda")
    for j in range(n):
        b.addcmul_(A[:, j, :], x[:, j:j + 1])
    return A, b


def _solve_inputs(case, seed):
    n, batch = case["n"], case["batch"]
    A, b = _systems(n, batch, _generator(seed))
    if case["layout"] == "soa":
        ld = batch + case["pad"]
        As = torch.zeros((n, n, ld), dtype=torch.float64, device="cuda")
        As[:, :, :batch] = A.permute(1, 2, 0)
        bs = torch.zeros((n, ld), dtype=torch.float64, device="cuda")
        bs[:, :batch] = b.t()
        A, b = As, bs
    return A, b


def _ragged_inputs(case, seed):
    g = _generator(seed)
    batch = case["batch"]
    # every size equally often, in an order of its own for each seed
    order = torch.randperm(batch, generator=g, device="cuda")
    n = (order % 31 + 2).to(torch.int32)
    n64 = n.to(torch.int64)
    offA = torch.cumsum(n64 * n64, 0) - n64 * n64
    offB = torch.cumsum(n64, 0) - n64
    A = torch.randn(int((n64 * n64).sum()), generator=g, dtype=torch.float64, device="cuda")
    b = torch.randn(int(n64.sum()), generator=g, dtype=torch.float64, device="cuda")
    return n, offA, offB, A, b


def _group_sizes(case):
    """The requests of a burst: their sizes belong to the case, their data to the seed."""
    g = torch.Generator()
    g.manual_seed(case["burst"])
    ns = torch.randint(2, 33, (case["groups"],), generator=g).tolist()
    us = torch.rand(case["groups"], generator=g, dtype=torch.float64).tolist()
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return [(n, int(round(math.exp(lo + (hi - lo) * u)))) for n, u in zip(ns, us)]


def _group_inputs(case, seed):
    g = _generator(seed)
    return [_systems(n, batch, g) for n, batch in _group_sizes(case)]


def _increments(case, seed):
    u = torch.rand((6, case["points"]), generator=_generator(seed), dtype=torch.float64,
                   device="cuda")
    return (u * 2 - 1) * case["amp"]


def _zeros(*shape, dtype=torch.int32):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    s = {"case": case, "ctx": lupp.lupp_create(torch.cuda.current_device())}
    kind = case["kind"]
    if kind == "solve":
        s["A0"], s["b0"] = _solve_inputs(case, seed)
        s["A"] = torch.empty_like(s["A0"]) if case["factors"] else s["A0"]
        s["b"] = torch.empty_like(s["b0"])
        aos = case["layout"] == "aos"
        n, batch = case["n"], case["batch"]
        s["ipiv"] = _zeros(batch, n) if aos else _zeros(n, batch + case["pad"])
        s["info"] = _zeros(batch)
    elif kind == "ragged":
        s["n"], s["offA"], s["offB"], s["A"], s["b0"] = _ragged_inputs(case, seed)
        s["b"] = torch.empty_like(s["b0"])
        s["ipiv"] = _zeros(s["b0"].numel())
        s["info"] = _zeros(case["batch"])
    elif kind == "grouped":
        data = _group_inputs(case, seed)
        total = sum(b.numel() for _, b in data)
        s["b0"] = torch.cat([b.reshape(-1) for _, b in data])
        s["b"], s["ipiv"] = torch.empty_like(s["b0"]), _zeros(total)
        s["info"] = _zeros(sum(A.shape[0] for A, _ in data))
        s["A"] = [A for A, _ in data]
        s["groups"], o, oi = [], 0, 0
        for A in s["A"]:
            batch, n = A.shape[0], A.shape[1]
            s["groups"].append(lupp.group(n, batch, A, s["b"][o:], s["ipiv"][o:], s["info"][oi:]))
            o, oi = o + batch * n, oi + batch
    else:
        law, count = case["law"], case["points"]
        s["deps"] = _increments(case, seed)
        s["state0"] = _zeros(law, count, dtype=torch.float64)
        s["state"] = torch.empty_like(s["state0"])
        s["sig"] = _zeros(6, count, dtype=torch.float64)
        s["iters"], s["status"] = _zeros(count), _zeros(count)
        s["tangent"] = _zeros(36, count, dtype=torch.float64) if case["tangent"] else None
        s["pts"] = lupp.points(s["deps"], s["state"], s["sig"], s["iters"], s["status"],
                               s["tangent"])
        s["law"] = lupp.make_law(law)
    return s


# -------------------------------------------------------------------- pass
def _ok(rc):
    if rc != 0:
        raise lupp.LuppError(rc, "pass")


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "newton":
        s["state"].copy_(s["state0"])
        _ok(lupp.constitutive_update(ctx, s["pts"], s["law"], 1e-12, 20))
        out = [s["sig"], s["state"], s["iters"], s["status"]]
        return out + [s["tangent"]] if case["tangent"] else out
    s["b"].copy_(s["b0"])
    if kind == "solve":
        n, batch, soa = case["n"], case["batch"], case["layout"] == "soa"
        flags = lupp.LUPP_FMA if case["fma"] else 0
        if case["factors"]:
            s["A"].copy_(s["A0"])
        else:
            flags |= lupp.LUPP_KEEP_A
        ld = batch + case["pad"]
        _ok(lupp.lupp_batched_solve(ctx, n, batch, lupp.LUPP_SOA if soa else lupp.LUPP_AOS,
                                    s["A"], n, ld if soa else n * n, s["b"], ld if soa else n,
                                    s["ipiv"], s["info"], flags))
        out = [s["b"], s["ipiv"], s["info"]]
        return out + [s["A"]] if case["factors"] else out
    if kind == "ragged":
        _ok(lupp.lupp_batched_solve_ragged(ctx, case["batch"], s["n"], s["offA"], s["offB"],
                                           s["A"], s["b"], s["ipiv"], s["info"],
                                           lupp.LUPP_KEEP_A))
    else:
        _ok(lupp.lupp_batched_solve_grouped(ctx, s["groups"], lupp.LUPP_KEEP_A))
    return [s["b"], s["ipiv"], s["info"]]


# -------------------------------------------------------------------- work
def _solve_flops(n):
    return sum(m + 2 * m * m for m in range(1, n)) + 2 * n * n - n


def _solve_bytes(n, factors):
    """Read A and b, write x, the int32 pivots and info, and the factors."""
    return (16 if factors else 8) * n * n + 20 * n + 4


def work(case):
    kind = case["kind"]
    if kind == "solve":
        n, batch = case["n"], case["batch"]
        return {"bytes": batch * _solve_bytes(n, case["factors"]), "flops": batch * _solve_flops(n)}
    sizes = range(2, 33)
    if kind == "ragged":
        per = case["batch"] / len(sizes)
        return {"bytes": int(per * sum(_solve_bytes(n, False) + 20 for n in sizes)),
                "flops": int(per * sum(_solve_flops(n) for n in sizes))}
    if kind == "grouped":
        burst = _group_sizes(case)
        return {"bytes": sum(batch * _solve_bytes(n, False) for n, batch in burst),
                "flops": sum(batch * _solve_flops(n) for n, batch in burst)}
    law, count = case["law"], case["points"]
    solves = SOLVES_PER_POINT * (1.0 if case["amp"] > 1e-3 else 0.5)
    # every iterate evaluates the residual and the Jacobian's entries once
    flops = solves * _solve_flops(law) + (solves + 1) * (4 * law * law + 10 * law)
    per_bytes = 8 * (6 + 2 * law + 6) + 8
    if case["tangent"]:
        flops += _solve_flops(law) + 5 * (2 * law * law - law)
        per_bytes += 36 * 8
    return {"bytes": count * per_bytes, "flops": int(count * flops)}


# ------------------------------------------------------------------- exact
def _lu_solve(a, rhs):
    """LU with partial pivoting of a (n, n, B), element (i, j) at [j][i], and
    the solutions of rhs (R, n, B). Overwrites both; returns ipiv, info."""
    n, B = a.shape[0], a.shape[2]
    ipiv = torch.empty((n, B), dtype=torch.int32, device=a.device)
    info = torch.zeros(B, dtype=torch.int32, device=a.device)
    for k in range(n):
        p = a[k, k:].abs().argmax(dim=0) + k
        ipiv[k] = (p + 1).to(torch.int32)
        for m in (a, rhs):
            at = p.expand(m.shape[0], 1, B)
            row = m.gather(1, at)
            m.scatter_(1, at, m[:, k:k + 1].clone())
            m[:, k:k + 1] = row
        zero = a[k, k] == 0
        info = torch.where(zero & (info == 0), torch.full_like(info, k + 1), info)
        if k + 1 < n:
            l = a[k, k + 1:] / a[k, k]
            a[k, k + 1:] = l
            a[k + 1:, k + 1:] -= l[None] * a[k + 1:, k][:, None]
            rhs[:, k + 1:] -= l[None] * rhs[:, k][:, None]
    for j in range(n - 1, -1, -1):
        rhs[:, j] /= a[j, j]
        if j:
            rhs[:, :j] -= a[j, :j][None] * rhs[:, j][:, None]
    return ipiv, info


def _chunks(total, n):
    step = max(1024, (1 << 26) // (n * n))
    for lo in range(0, total, step):
        yield lo, min(total, lo + step)


def _exact_packed(A, b):
    """x, ipiv, info and factors of packed systems A (batch, n, n), b (batch, n)."""
    batch, n = b.shape
    x, lu = torch.empty_like(b), torch.empty_like(A)
    ipiv, info = _zeros(batch, n), _zeros(batch)
    for lo, hi in _chunks(batch, n):
        a = A[lo:hi].permute(1, 2, 0).contiguous()
        r = b[lo:hi].t().contiguous()[None]
        ip, inf = _lu_solve(a, r)
        x[lo:hi], lu[lo:hi] = r[0].t(), a.permute(2, 0, 1)
        ipiv[lo:hi], info[lo:hi] = ip.t(), inf
    return x, ipiv, info, lu


def _exact_solve(case, seed):
    A, b = _solve_inputs(case, seed)
    n, batch = case["n"], case["batch"]
    if case["layout"] == "aos":
        x, ipiv, info, lu = _exact_packed(A, b)
    else:
        x, lu = b.clone(), A.clone()
        ipiv, info = _zeros(n, batch + case["pad"]), _zeros(batch)
        for lo, hi in _chunks(batch, n):
            a = A[:, :, lo:hi].contiguous()
            r = b[:, lo:hi].contiguous()[None]
            ipiv[:, lo:hi], info[lo:hi] = _lu_solve(a, r)
            x[:, lo:hi], lu[:, :, lo:hi] = r[0], a
    return [x, ipiv, info, lu] if case["factors"] else [x, ipiv, info]


def _exact_ragged(case, seed):
    n, offA, offB, A, b = _ragged_inputs(case, seed)
    x, ipiv, info = torch.empty_like(b), _zeros(b.numel()), _zeros(case["batch"])
    for m in range(2, 33):
        idx = torch.nonzero(n == m)[:, 0]
        if idx.numel() == 0:
            continue
        ia = offA[idx][:, None] + torch.arange(m * m, device="cuda")
        ib = offB[idx][:, None] + torch.arange(m, device="cuda")
        xs, ip, inf, _ = _exact_packed(A[ia].view(-1, m, m), b[ib])
        x[ib], ipiv[ib], info[idx] = xs, ip, inf
    return [x, ipiv, info]


def _exact_grouped(case, seed):
    parts = [_exact_packed(A, b) for A, b in _group_inputs(case, seed)]
    return [torch.cat([p[i].reshape(-1) for p in parts]) for i in range(3)]


class _Norton:
    """The material and time step of lupp.make_law's defaults."""
    E, nu, A, m, C, D, dt = 200e3, 0.3, 1e-8, 5.0, 1e4, 100.0, 1e-2


def _law(kind, de, y):
    """Residual F (kind, B), Jacobian J (kind, kind, B) as [column][row] and
    stress of the Norton law (7) or Norton + Armstrong-Frederick (13) from a
    virgin state, as written in the interface header."""
    L, B = _Norton, de.shape[1]
    lam = L.E * L.nu / ((1 + L.nu) * (1 - 2 * L.nu))
    mu2 = L.E / (1 + L.nu)
    af = kind == 13
    e, dp = y[:6], y[6]
    one = torch.zeros((6, 1), dtype=torch.float64, device=de.device)
    one[:3] = 1
    sig = mu2 * e + lam * e[:3].sum(0) * one
    c = 2.0 / 3.0 * L.C if af else 0.0
    xi = sig - one * (sig[:3].sum(0) / 3)
    if af:
        xi = xi - c * y[7:]
    seq = torch.sqrt(1.5 * (xi * xi).sum(0))
    on = seq > 0
    safe = torch.where(on, seq, torch.ones_like(seq))
    N = torch.where(on, 1.5 * xi / safe, torch.zeros_like(xi))
    I6 = torch.eye(6, dtype=torch.float64, device=de.device)[:, :, None]
    G = torch.where(on, (1.5 * I6 - N[:, None] * N[None]) / safe, torch.zeros_like(seq))
    P = torch.eye(6, dtype=torch.float64, device=de.device) - one @ one.t() / 3
    GK = torch.einsum("abp,bc->acp", G, P)
    rate = L.dt * L.A
    F = torch.empty((kind, B), dtype=torch.float64, device=de.device)
    J = torch.zeros((kind, kind, B), dtype=torch.float64, device=de.device)  # [row][column]
    F[:6] = e + dp * N - de
    F[6] = dp - rate * seq ** L.m
    g = rate * L.m * seq ** (L.m - 1) * on
    J[:6, :6] = I6 + dp * mu2 * GK
    J[:6, 6] = N
    J[6, :6] = -g * mu2 * torch.einsum("ab,bp->ap", P, N)
    J[6, 6] = 1
    if af:
        al = y[7:]
        F[7:] = al - dp * N + L.D * dp * al
        J[:6, 7:] = -c * dp * G
        J[6, 7:] = c * g * N
        J[7:, :6] = -mu2 * dp * GK
        J[7:, 6] = -N + L.D * al
        J[7:, 7:] = I6 * (1 + L.D * dp) + c * dp * G
    return F, J.transpose(0, 1).contiguous(), sig, mu2, lam


def _exact_newton(case, seed):
    kind, count = case["law"], case["points"]
    de_all = _increments(case, seed)
    state = _zeros(kind, count, dtype=torch.float64)
    sigs = _zeros(6, count, dtype=torch.float64)
    its, sts = _zeros(count), _zeros(count)
    tan = _zeros(36, count, dtype=torch.float64)
    for lo, hi in _chunks(count, kind):
        de = de_all[:, lo:hi]
        y = torch.zeros((kind, hi - lo), dtype=torch.float64, device="cuda")
        live = torch.ones(hi - lo, dtype=torch.bool, device="cuda")
        it = torch.zeros(hi - lo, dtype=torch.int32, device="cuda")
        st = torch.ones_like(it)
        for k in range(21):
            F, J, _, _, _ = _law(kind, de, y)
            ok = F.abs().amax(0) < 1e-12
            st[live & ok] = 0
            live &= ~ok
            if k == 20 or not bool(live.any()):
                break
            r = (-F)[None].clone()
            _lu_solve(J, r)
            y = torch.where(live, y + r[0], y)
            it += live.to(torch.int32)
        F, J, sig, mu2, lam = _law(kind, de, y)
        done = st == 0
        sigs[:, lo:hi], its[lo:hi], sts[lo:hi] = sig, it, st
        state[:, lo:hi] = torch.where(done, y, torch.zeros_like(y))
        if case["tangent"]:
            R = torch.zeros((6, kind, hi - lo), dtype=torch.float64, device="cuda")
            for c in range(6):
                R[c, c] = 1
            _lu_solve(J, R)
            t = mu2 * R[:, :6]
            t[:, :3] += lam * R[:, :3].sum(1, keepdim=True)
            t = t.permute(1, 0, 2).reshape(36, hi - lo)
            tan[:, lo:hi] = torch.where(done, t, torch.zeros_like(t))
    out = [sigs, state, its, sts]
    return out + [tan] if case["tangent"] else out


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        return _exact_solve(case, seed)
    if kind == "ragged":
        return _exact_ragged(case, seed)
    if kind == "grouped":
        return _exact_grouped(case, seed)
    return _exact_newton(case, seed)
