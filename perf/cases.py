"""What users of the library run, as cases to be timed and compared.

A case is one pass of a user's program: vertex configurations in hand on the
GPU, propagators built from them, then connected sums or their gradients,
through the Python entry points.  The listed cases cover orders 4 to 12, one
configuration to thousands, one to six flavour slots, forward and reverse, the
labelled (bipartite) form, the mask-only form and reproducible gradients.
``draw`` gives further cases of the same ranges.

The reference values (``exact``) come from a dynamic programme over
(visited counts, head, current) states in plain torch float64, whole levels at
a time, differentiated by torch.autograd where gradients are asked for.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2507_12349_amd import _binding as B
from paper_2507_12349_amd.autograd import ConnectedSum, G0Propagator, Geometry
from paper_2507_12349_amd.workloads import Draw, Workload

F64 = torch.float64


def _case(name, kind, n, nconf, nflav, variant, L, beta, **more):
    c = dict(kind=kind, n=n, n_hi=more.pop("n_hi", n), nconf=nconf, nflav=nflav, variant=variant, L=L, beta=beta,
             stubs=False, mask_only=False, deterministic=False)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one configuration of low order: a caller that evaluates diagrams one
        # at a time (the 4x4 SU(2) single-configuration workload); all latency
        _case("single_n4", "forward", 4, 1, 2, B.UNIFORM, 4, 2.0),
        # one batch of the Monte Carlo series at a low order: sample, propagators,
        # sums, moments (the series loop's 8192 samples per batch on 8x8)
        _case("series_n5", "series", 5, 8192, 4, B.UNIFORM, 8, 4.0),
        # gradient in chemical potentials and shifts at low order, a ragged batch,
        # three flavours of their own (fits of shift parameters)
        _case("shift_gradient_n6", "gradient", 6, 333, 3, B.FLAVOUR, 8, 4.0, stubs=True),
        # the 4096-configuration SU(4) batch of order 8
        _case("batch_n8", "forward", 8, 4096, 4, B.UNIFORM, 8, 4.0),
        # one optimisation step through torch.autograd, from (mu, alpha) to a loss
        _case("autograd_n8", "autograd", 8, 1000, 4, B.UNIFORM, 8, 4.0),
        # the headline step: 2048 configurations of order 10, SU(4), propagators,
        # reverse sweep and chain rule to (mu, shift)
        _case("gradient_n10", "gradient", 10, 2048, 4, B.UNIFORM, 8, 4.0, stubs=True),
        # broken symmetry: three flavour matrices, order 10, forward sums
        _case("sym_broken_n10", "forward", 10, 1024, 3, B.FLAVOUR, 8, 4.0),
        # mixed orders 6..12 of a series, six flavours with shift heads, 16x16
        _case("uneven_n6_12", "forward", 6, 600, 6, B.FLAVOUR, 16, 5.0, n_hi=12, stubs=True),
        # honeycomb lattice, labels summed, SU(2) with a staggered field, order 8
        _case("honeycomb_n8", "honeycomb", 8, 1024, 2, B.FLAVOUR, 16, 5.0),
        # the same with gradients, one order lower, a ragged batch
        _case("honeycomb_gradient_n7", "honeycomb_gradient", 7, 600, 2, B.FLAVOUR, 16, 5.0),
        # SU(2) without cycle factors (mask-only states), forward and reverse
        _case("mask_only_n10", "gradient", 10, 1024, 2, B.FLAVOUR, 8, 4.0, mask_only=True),
        # gradients that repeat bit for bit
        _case("reproducible_n9", "gradient", 9, 1024, 4, B.UNIFORM, 8, 4.0, deterministic=True),
    ]


_COST_MAX = 1.2e11   # bytes of states a drawn case may pass over (the largest listed case's)
_PAD = 64            # configurations run in groups of this many


def _cost(c):
    """A rough size of a case: states times the times each is read or written."""
    pad = -(-c["nconf"] // _PAD) * _PAD
    nmat = c["nflav"] if c["variant"] == B.FLAVOUR else 1
    if c["kind"].startswith("honeycomb"):
        s = B.plan_counts_sublattice(c["n"])["states"]
    else:
        s = max(B.plan_counts(k)["states"] for k in range(c["n"], c["n_hi"] + 1))
    passes = 16 if c["kind"] in ("forward", "series", "honeycomb") else 48
    if c["deterministic"]:
        passes *= 3
    return float(s) * pad * nmat * passes


def draw(rng):
    kind = rng.choice(["forward"] * 4 + ["series"] * 2 + ["gradient"] * 5 + ["autograd", "honeycomb", "honeycomb",
                                                                             "honeycomb_gradient"])
    while True:
        L, beta = rng.choice([4, 6, 8, 12, 16]), round(rng.uniform(2.0, 5.0), 2)
        nconf = int(round(math.exp(rng.uniform(0.0, math.log(8192.0)))))
        if kind.startswith("honeycomb"):
            c = _case("", kind, rng.randint(3, 8), min(nconf, 2048), 2, B.FLAVOUR, L, beta)
        elif kind == "series":
            c = _case("", kind, rng.randint(3, 8), max(nconf, 500), rng.choice([2, 3, 4]), B.UNIFORM, rng.choice([4, 8]),
                      beta)
        elif kind == "autograd":
            c = _case("", kind, rng.randint(4, 9), nconf, rng.choice([2, 4]), B.UNIFORM, L, beta)
        else:
            variant = rng.choice([B.UNIFORM, B.FLAVOUR])
            nflav = rng.randint(2, 6)
            c = _case("", kind, rng.randint(3, 11), nconf, nflav, variant, L, beta, stubs=rng.random() < 0.4)
            what = rng.random()
            if kind == "forward" and what < 0.2:
                c["n_hi"] = min(11, c["n"] + rng.randint(1, 5))
            elif kind == "gradient" and what < 0.15:
                c["deterministic"] = True
            elif what > 0.85:
                c.update(variant=B.FLAVOUR, nflav=2, stubs=False, mask_only=True)
        if _cost(c) <= _COST_MAX:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_U = 1.0


def _inputs(c, seed):
    """Host inputs of a case: orders, sites, times, potentials, shifts, weights."""
    rng = np.random.default_rng([int(seed), 2507])
    nmat = c["nflav"] if c["variant"] == B.FLAVOUR else 1
    # the orders belong to the case (the plan), everything else to the seed
    n = np.random.default_rng([c["nconf"], c["n"], c["n_hi"]]).integers(c["n"], c["n_hi"] + 1, size=c["nconf"])
    n = n.astype(np.int32)
    tot = int(n.sum())
    site = rng.integers(0, c["L"] ** 2, size=tot)
    sites = np.stack([site % c["L"], site // c["L"]], axis=1).astype(np.int32)
    tau = rng.uniform(0.0, c["beta"], size=tot)
    mu = -0.5 + rng.uniform(-0.3, 0.3, size=nmat)
    alpha = rng.uniform(-0.2, 0.2, size=nmat) if c["stubs"] else np.zeros(nmat)
    delta = 0.3 * (1.0 - 2.0 * (np.arange(nmat) % 2))
    obar = rng.normal(size=c["nconf"])
    return dict(nmat=nmat, n=n, sites=sites, tau=tau, mu=mu, alpha=alpha, delta=delta, obar=obar, seed=int(seed))


def _draw_of(c, x):
    w = Workload(c["kind"], L=c["L"], t=1.0, beta=c["beta"], nflav=c["nflav"], variant=c["variant"],
                 mu=tuple(x["mu"]), n=c["n"], nconf=c["nconf"], seed=0, stubs=c["stubs"], U=_U)
    voff = np.zeros(c["nconf"], dtype=np.int64)
    voff[1:] = np.cumsum(x["n"][:-1], dtype=np.int64)
    return Draw(w, x["n"], voff, x["sites"], x["tau"], x["alpha"])


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    nc, nmat = c["nconf"], x["nmat"]
    sub = c["kind"].startswith("honeycomb")
    geo = Geometry(_draw_of(c, x), nmat, sublattice=sub)
    dev = geo.device
    s = dict(c=c, x=x, geo=geo)
    s["batch"] = B.Batch(x["n"], c["nflav"], c["variant"], stubs=c["stubs"], sublattice=sub,
                         mask_only=c["mask_only"], deterministic=c["deterministic"])
    s["stub"] = torch.as_tensor(np.tile(x["alpha"] / _U, (nc, 1)), device=dev) if c["stubs"] else None
    if c["kind"] == "autograd":
        s["mu"] = torch.tensor(x["mu"], dtype=F64, requires_grad=True)
        s["alpha"] = torch.tensor(x["alpha"], dtype=F64, requires_grad=True)
        s["weight"] = torch.as_tensor(x["obar"], device=dev)
        return s
    s["S"] = torch.empty(nc, dtype=F64, device=dev)
    s["G"] = torch.empty(geo.total, dtype=F64, device=dev)
    if c["kind"] == "series":
        s["sites"] = torch.empty((nc * c["n"], 2), dtype=torch.int32, device=dev)
        s["tau"] = torch.empty(nc * c["n"], dtype=F64, device=dev)
    if c["kind"] in ("gradient", "honeycomb_gradient"):
        s["dG"], s["G_bar"] = torch.empty_like(s["G"]), torch.empty_like(s["G"])
        s["stub_bar"] = None if s["stub"] is None else torch.empty_like(s["stub"])
        s["obar"] = torch.as_tensor(x["obar"], device=dev)
        s["mu_bar"], s["alpha_bar"] = (torch.empty(nc * nmat, dtype=F64, device=dev) for _ in range(2))
    return s


def run(state):
    s = state
    c, x, geo, b = s["c"], s["x"], s["geo"], s["batch"]
    if c["kind"] == "autograd":
        s["mu"].grad = s["alpha"].grad = None
        S = ConnectedSum.apply(G0Propagator.apply(s["mu"], s["alpha"], geo), None, b, geo.Goff, -1.0)
        (S * s["weight"]).sum().backward()
        return dict(S=S, mu=s["mu"].grad, alpha=s["alpha"].grad)
    if c["kind"] == "series":
        acc = torch.zeros(2, dtype=F64, device=geo.device)
        B.mc_sample(geo.nconf, c["n"], geo.L, geo.beta, x["seed"], 0, s["sites"], s["tau"])
        B.build_g0(geo.nconf, geo.n, geo.voff, s["sites"], s["tau"], geo.L, geo.t, geo.beta, x["mu"], x["alpha"],
                   geo.Goff, s["G"], None)
        b.forward(s["G"], geo.Goff, None, -1.0, s["S"])
        B.accumulate_moments(geo.nconf, s["S"], acc)
        return dict(S=s["S"], moments=acc)
    dG = s.get("dG")
    if c["kind"].startswith("honeycomb"):
        B.build_g0_honeycomb(geo.nconf, geo.n, geo.voff, geo.sites, geo.tau, geo.L, geo.t, geo.beta, x["mu"],
                             x["alpha"], x["delta"], geo.Goff, s["G"], dG=dG)
    else:
        B.build_g0(geo.nconf, geo.n, geo.voff, geo.sites, geo.tau, geo.L, geo.t, geo.beta, x["mu"], x["alpha"],
                   geo.Goff, s["G"], dG)
    if dG is None:
        b.forward(s["G"], geo.Goff, s["stub"], -1.0, s["S"])
        return dict(G=s["G"], S=s["S"])
    b.adjoint(s["G"], geo.Goff, s["stub"], -1.0, s["obar"], s["S"], s["G_bar"], s["stub_bar"])
    B.chain_mu_shift(geo.nconf, geo.side, x["nmat"], geo.Goff, s["G_bar"], dG, s["stub_bar"],
                     1 if s["stub"] is None else x["nmat"], _U, s["mu_bar"], s["alpha_bar"])
    return dict(G=s["G"], S=s["S"], G_bar=s["G_bar"], stub_bar=s["stub_bar"], mu_bar=s["mu_bar"],
                alpha_bar=s["alpha_bar"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Inputs read once and outputs written once; two operations per transition
    and close of the dynamic programme and flavour (three times that with
    gradients), and about ten per exponential of a propagator."""
    c = case
    nmat = c["nflav"] if c["variant"] == B.FLAVOUR else 1
    sub = c["kind"].startswith("honeycomb")
    grad = c["kind"] in ("gradient", "honeycomb_gradient", "autograd")
    byts = flops = 0.0
    orders = range(c["n"], c["n_hi"] + 1)
    for n in orders:
        side = 2 * n if sub else n
        p = (B.plan_counts_mask_only(n) if c["mask_only"] else B.plan_counts_sublattice(n) if sub else B.plan_counts(n))
        step = 2.0 * (p["ext"] + p["closes"]) * (1 if c["mask_only"] else nmat)
        byts += 16 * n + 8 * nmat * side * side * (3 if grad else 1) + 8
        flops += step * (3 if grad else 1) + 10.0 * nmat * n * n * c["L"] ** 2 * (2 if sub else 1)
    per = c["nconf"] / len(orders)
    return {"bytes": byts * per, "flops": flops * per}


# ---------------------------------------------------------------------------
# reference values in plain torch float64
# ---------------------------------------------------------------------------
def _levels(n):
    """Rows (visited counts m, head u) by level: row (m, 0) for m_0 >= 1 and
    (m, u) for m_0 = m_u = 2, and where each extension leads."""
    p3 = 3 ** np.arange(n)
    dig = (np.arange(3 ** n)[:, None] // p3) % 3
    rows = dig[:, :1].repeat(n, 1) >= 1
    rows[:, 1:] = (dig[:, :1] == 2) & (dig[:, 1:] == 2)
    level = dig.sum(1)
    idx = np.full((3 ** n, n), -1, dtype=np.int64)
    per = []
    for l in range(1, 2 * n + 1):
        code, u = np.nonzero(rows & (level == l)[:, None])
        idx[code, u] = np.arange(code.size)
        per.append((code, u))
    dev = torch.device("cuda")
    out = []
    for code, u in per:
        ext = []
        for w in range(n):
            sel = np.nonzero(dig[code, w] < 2)[0]
            child = idx[code[sel] + p3[w], u[sel]]
            fac = np.where(dig[code[sel], w] == 0, 2.0, 1.0)
            sh = np.where(dig[code[sel], w] == 1, np.where(code[sel] == 1, 2.0, 1.0), 0.0)
            ext.append([torch.as_tensor(v, device=dev) for v in (sel, child, fac, sh)])
        masks, inv = np.unique(code, return_inverse=True)
        one = dig[masks] == 1
        has = np.nonzero(one.any(1))[0]
        h = one[has].argmax(1)
        cl = [torch.as_tensor(v, device=dev) for v in (inv, has, h, idx[masks[has] + p3[h], h])]
        out.append((code.size, masks.size, torch.as_tensor(u, device=dev), ext, cl))
    return out


def _sums(plan, n, G, nflav, variant, sig):
    """Connected sums of a stack of configurations: G [b, nmat, n, n], sig [b, nmat] or None."""
    b, nmat = G.shape[:2]
    W = -float(nflav) if variant == B.UNIFORM else -1.0
    Gf = G.reshape(b * nmat, n, n)
    F = torch.zeros(b * nmat, 1, n, dtype=F64, device=G.device)
    F[:, 0, 0] = 1.0
    for i, (nr, nm, u, ext, (inv, has, h, crow)) in enumerate(plan):
        acc = torch.bmm(F, Gf)
        close = acc.gather(2, u.view(1, nr, 1).expand(b * nmat, nr, 1)).view(b, nmat, nr).sum(1)
        t = W * torch.zeros(b, nm, dtype=F64, device=G.device).index_add(1, inv, close)
        if i == len(plan) - 1:
            return t[:, 0]
        nxt, cols = plan[i + 1][0], []
        for w in range(n):
            sel, child, fac, sh = ext[w]
            val = acc[:, :, w].index_select(1, sel) * fac
            if sig is not None:
                val = val - F[:, :, w].index_select(1, sel) * sh * sig.reshape(b * nmat, 1)
            col = torch.zeros(b * nmat, nxt, dtype=F64, device=G.device).index_copy(1, child, val)
            at = torch.nonzero(h == w)[:, 0]
            op = t.index_select(1, has.index_select(0, at)).repeat_interleave(nmat, 0)
            cols.append(col.index_add(1, crow.index_select(0, at), op))
        F = torch.stack(cols, 2)


def _square_g0(sites, tau, L, beta, xi0):
    """G [b, nmat, n, n] on the square lattice; xi0 [b, nmat] = alpha - mu."""
    k = 2.0 * math.pi * torch.arange(L, dtype=F64, device=tau.device) / L
    eps = (-2.0 * (torch.cos(k)[:, None] + torch.cos(k)[None, :])).reshape(-1)
    dx = sites[:, :, None, :] - sites[:, None, :, :]
    m = torch.arange(L * L, device=tau.device)
    ph = ((m // L) * dx[..., :1] + (m % L) * dx[..., 1:]) % L
    cosk = torch.cos(2.0 * math.pi * ph.to(F64) / L)                  # [b, n, n, L^2]
    d = (tau[:, :, None] - tau[:, None, :])[..., None]
    out = []
    for g in range(xi0.shape[1]):
        xi = (eps + xi0[:, g, None])[:, None, None, :]
        out.append((cosk * _branch(xi, d, beta)).mean(-1))
    return torch.stack(out, 1)


def _branch(x, d, beta):
    """-e^{-x d} (1 - n_F) for d > 0 and e^{-x d} n_F for d <= 0, exponents kept non-positive."""
    fwd, pos = d > 0, x >= 0
    c = torch.where(fwd, torch.where(pos, -d, beta - d), torch.where(pos, -(beta + d), -d))
    return torch.where(fwd, -1.0, 1.0) * torch.exp(x * c) / (1.0 + torch.exp(-beta * x.abs()))


def _honeycomb_g0(cells, tau, L, beta, xi0, delta):
    """G [b, nmat, 2n, 2n] on the honeycomb lattice, index 2k + s."""
    b, n = tau.shape
    dev = tau.device
    m = torch.arange(L * L, device=dev)
    k1, k2 = (2.0 * math.pi * v.to(F64) / L for v in (m % L, m // L))
    er, ei = -(1.0 + torch.cos(k1) + torch.cos(k2)), -(torch.sin(k1) + torch.sin(k2))
    dr = cells[:, :, None, :] - cells[:, None, :, :]
    ph = 2.0 * math.pi * (((m % L) * dr[..., :1] + (m // L) * dr[..., 1:]) % L).to(F64) / L
    d = (tau[:, :, None] - tau[:, None, :])[..., None]
    out = []
    for g in range(xi0.shape[1]):
        dz = float(delta[g])
        r = torch.sqrt(er * er + ei * ei + dz * dz)
        x = xi0[:, g].view(b, 1, 1, 1)
        fp, fm = _branch(x + r, d, beta), _branch(x - r, d, beta)
        S, D = 0.5 * (fp + fm), 0.5 * (fp - fm) / r
        c, s = torch.cos(ph), torch.sin(ph)
        aa, bb = (c * (S + D * dz)).mean(-1), (c * (S - D * dz)).mean(-1)
        ab, ba = (D * (c * er - s * ei)).mean(-1), (D * (c * er + s * ei)).mean(-1)
        out.append(torch.stack([torch.stack([aa, ab], -1), torch.stack([ba, bb], -1)], 3)
                   .permute(0, 1, 3, 2, 4).reshape(b, 2 * n, 2 * n))
    return torch.stack(out, 1)


def _splitmix(ctr, seed):
    with np.errstate(over="ignore"):
        z = np.uint64(seed & 0xFFFFFFFFFFFFFFFF) + np.uint64(0x9E3779B97F4A7C15) * (ctr + np.uint64(1))
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _sampled(c, seed):
    """Sites and times of the series' sampler (vertex 0 at the origin)."""
    i = np.arange(c["nconf"] * c["n"], dtype=np.uint64)
    site = ((_splitmix(2 * i, seed) >> np.uint64(32)) * np.uint64(c["L"] ** 2)) >> np.uint64(32)
    tau = c["beta"] * ((_splitmix(2 * i + 1, seed) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53)
    sites = np.stack([site % c["L"], site // c["L"]], axis=1).astype(np.int32)
    sites[:: c["n"]], tau[:: c["n"]] = 0, 0.0
    return sites, tau


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    sub = c["kind"].startswith("honeycomb")
    grad = c["kind"] in ("gradient", "honeycomb_gradient", "autograd")
    if sub and (2 ** c["n"] * c["nconf"] > 3e5 or (grad and 2 ** c["n"] * c["nconf"] > 1e5)):
        return None   # more label assignments than there is time for
    if c["kind"] == "series":
        x["sites"], x["tau"] = _sampled(c, x["seed"])
    dev, nmat = torch.device("cuda"), x["nmat"]
    voff = np.concatenate([[0], np.cumsum(x["n"])])
    nc = c["nconf"]
    xi0 = torch.as_tensor(np.tile(x["alpha"] - x["mu"], (nc, 1)), device=dev)
    sig = torch.as_tensor(np.tile(x["alpha"] / _U, (nc, 1)), device=dev) if c["stubs"] else None
    obar = torch.as_tensor(x["obar"], device=dev)
    S = torch.empty(nc, dtype=F64, device=dev)
    Gs, Gb = [None] * nc, [None] * nc
    xb, sb = torch.zeros(nc, nmat, dtype=F64, device=dev), torch.zeros(nc, nmat, dtype=F64, device=dev)
    for n in sorted(set(x["n"].tolist())):
        plan = _levels(n)
        which = np.nonzero(x["n"] == n)[0]
        # stacks that fit the card: the widest level forward, every level with gradients
        rows = sum(p[0] for p in plan) * 6 if grad else max(p[0] for p in plan) * 8
        step = max(1, int(6e10 / (8.0 * rows * n * nmat * (2 ** n if sub else 1))))
        for a in range(0, which.size, step):
            at = which[a:a + step]
            ti = torch.as_tensor(at, device=dev)
            vs = voff[at][:, None] + np.arange(n)
            sites = torch.as_tensor(x["sites"][vs], device=dev).long()
            tau = torch.as_tensor(x["tau"][vs], device=dev)
            x0 = xi0[ti].requires_grad_(grad)
            sg = sig[ti].requires_grad_(grad) if sig is not None else None
            with torch.set_grad_enabled(grad):
                if sub:
                    G = _honeycomb_g0(sites, tau, c["L"], c["beta"], x0, x["delta"])
                    lab = (torch.arange(2 ** n, device=dev)[:, None] >> torch.arange(n, device=dev)) & 1
                    pick = 2 * torch.arange(n, device=dev) + lab                    # [2^n, n]
                    Gl = G[:, :, pick[:, :, None], pick[:, None, :]]                # [b, nmat, 2^n, n, n]
                    Gl = Gl.permute(0, 2, 1, 3, 4).reshape(-1, nmat, n, n)
                    s = _sums(plan, n, Gl, c["nflav"], c["variant"], None).view(at.size, -1).sum(1)
                else:
                    G = _square_g0(sites, tau, c["L"], c["beta"], x0)
                    s = _sums(plan, n, G, c["nflav"], c["variant"], sg)
                if c["mask_only"]:
                    s = s * 0.5 ** n
            S[ti] = s.detach()
            if grad:
                gr = torch.autograd.grad((s * obar[ti]).sum(), [G, x0] + ([sg] if sg is not None else []))
                xb[ti] = gr[1]
                if sg is not None:
                    sb[ti] = gr[2]
            for i, k in enumerate(at):
                Gs[k] = G[i].detach().reshape(-1)
                Gb[k] = gr[0][i].reshape(-1) if grad else None
            del G, s
    if c["kind"] == "autograd":
        return dict(S=S, mu=-xb.sum(0), alpha=xb.sum(0))
    if c["kind"] == "series":
        return dict(S=S, moments=torch.stack([S.sum(), (S * S).sum()]))
    out = dict(G=torch.cat(Gs), S=S)
    if grad:
        out.update(G_bar=torch.cat(Gb), stub_bar=sb if sig is not None else None, mu_bar=-xb.reshape(-1),
                   alpha_bar=(xb + sb / _U).reshape(-1))
    return out
