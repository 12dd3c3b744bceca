"""Benchmark: connected-sum configurations per second at n = 10, SU(4), FP64.

One step = the whole hot path over one batch of 2048 synthetic vertex
configurations (8x8 lattice, beta = 4, mu = -0.5, uniform SU(4), shifts at
delta = 0), inputs resident on the GPU:
  propagators (G0 kernel)  ->  reverse sweep (the forward sum is recomputed
  inside and S is written)  ->  chain rule to (mu, shift).
`value` = configurations per second of that step (forward + adjoint).
Also reported: the batched forward alone (G0 + forward) and the plain form
(one launch per configuration, forward only) on the same device.

Prints ONE JSON line.  Options: --gpus (only 1 is supported), --steps,
--warmup, --no-cpu (skip the oracle baseline), --nconf.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP64 = 78.6e12           # MI355X FP64 vector peak, FLOP/s
PEAK_HBM = 8.0e12             # MI355X HBM3E, bytes/s
REV_KERNEL = "level_adj_kernel<%d, false, false>"
WORKLOAD = "adjoint"


def _kernel_hash():
    """Hash of the sources that define the unlabelled level kernels (whose HBM
    counters profiles/traffic.json holds) and their launches."""
    h = hashlib.sha256()
    for f in ("cos_level.hip", "libcos.cpp", "cos_internal.hpp", "cos_device.hpp"):
        with open(os.path.join(ROOT, "paper_2507_12349_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _traffic(kernel):
    """HBM bytes per launch from committed rocprofv3 counter runs, if they were
    taken on the current kernel sources; else None."""
    p = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(p):
        return None
    with open(p) as f:
        t = json.load(f)
    if t.get("kernel_sources_sha") != _kernel_hash():
        return None
    e = t.get("kernels", {}).get(kernel)
    return None if e is None else e.get("bytes_per_launch")


def honeycomb_forward(B, torch, reps):
    """Second workload (bipartite lattice, sublattice labels summed): honeycomb
    propagators + labelled forward levels over 1024 configurations of n = 8,
    two flavours; inputs resident on the device, launch shape autotuned."""
    from paper_2507_12349_amd.workloads import draw
    d = draw("honeycomb")
    w = d.workload
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    n = d.n.astype(np.int64)
    sizes = w.nflav * (2 * n) ** 2
    off = np.zeros(n.size, dtype=np.int64)
    off[1:] = np.cumsum(sizes[:-1])
    G = torch.empty(int(sizes.sum()), dtype=torch.float64, device=dev)
    Goff = torch.as_tensor(off, device=dev)
    dn, dv = torch.as_tensor(d.n, device=dev), torch.as_tensor(d.voff, device=dev)
    dc, dt = torch.as_tensor(d.sites, device=dev), torch.as_tensor(d.tau, device=dev)
    mu, al, st = np.array(w.mu), np.zeros(w.nflav), np.array(w.stagger)
    b = B.Batch(d.n, w.nflav, 1, sublattice=True)
    S = torch.empty(n.size, dtype=torch.float64, device=dev)

    def g0():
        B.build_g0_honeycomb(n.size, dn, dv, dc, dt, w.L, w.t, w.beta, mu, al, st, Goff, G, stream)

    g0()
    b.autotune(G, Goff, None, -1.0, S, stream=stream)
    b.forward(G, Goff, None, -1.0, S, stream)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    b.timing(True)
    e0.record(stream)
    for _ in range(reps):
        g0()
        b.forward(G, Goff, None, -1.0, S, stream)
    e1.record(stream)
    torch.cuda.synchronize()
    ph, _ = b.timing_read()
    b.timing(False)
    ms = e0.elapsed_time(e1) / reps
    fwd_ms = ph["forward"] / reps
    nn = int(n[0])
    pc = B.plan_counts_sublattice(nn)
    flop = w.nflav * 2.0 * (pc["ext"] + pc["closes"])          # per configuration
    states_bytes = w.nflav * 16.0 * pc["states"]                # each state written once, read once
    shape = b.launch_shape(nn)
    b.close()
    # the same sum by the mask-only variant (Alg. 1 with its labels)
    bm = B.Batch(d.n, w.nflav, 1, sublattice=True, mask_only=True)
    Sm = torch.empty_like(S)
    bm.autotune(G, Goff, None, -1.0, Sm, stream=stream)
    torch.cuda.synchronize()
    m0, m1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    m0.record(stream)
    for _ in range(reps):
        bm.forward(G, Goff, None, -1.0, Sm, stream)
    m1.record(stream)
    torch.cuda.synchronize()
    bm.close()
    ref = S / float(2 ** nn)
    # gradient step: propagators and dG/dxi -> labelled reverse sweep -> chain rule to (mu, alpha)
    dG = torch.empty_like(G)
    side = torch.as_tensor(2 * d.n, device=dev)
    ba = B.Batch(d.n, w.nflav, 1, sublattice=True)
    ob = torch.ones(n.size, dtype=torch.float64, device=dev)
    Sg, Gb = torch.empty_like(S), torch.empty_like(G)
    mub = torch.empty(n.size * w.nflav, dtype=torch.float64, device=dev)
    alb = torch.empty_like(mub)

    def grad_step():
        B.build_g0_honeycomb(n.size, dn, dv, dc, dt, w.L, w.t, w.beta, mu, al, st, Goff, G, stream, dG=dG)
        ba.adjoint(G, Goff, None, -1.0, ob, Sg, Gb, None, stream)
        B.chain_mu_shift(n.size, side, w.nflav, Goff, Gb, dG, None, 1, 1.0, mub, alb, stream)

    grad_step()
    ba.autotune(G, Goff, None, -1.0, Sg, ob, Gb, None, stream=stream)
    grad_step()
    torch.cuda.synchronize()
    a0, a1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ba.timing(True)
    a0.record(stream)
    for _ in range(reps):
        grad_step()
    a1.record(stream)
    torch.cuda.synchronize()
    aph, _ = ba.timing_read()
    ba.timing(False)
    grad = {"configs_per_s": n.size / (a0.elapsed_time(a1) / reps * 1e-3),
            "ms_per_step": a0.elapsed_time(a1) / reps,
            "phases_ms": {k: v / reps for k, v in aph.items()},
            "kernel": "sub_adj_kernel<8, true, false>", "launch_shape": ba.launch_shape(nn),
            "S_equals_forward": bool(torch.equal(Sg, S))}
    ba.close()
    mask_only = {"forward_levels_ms": m0.elapsed_time(m1) / reps,
                 "configs_per_s_forward_levels": n.size / (m0.elapsed_time(m1) / reps * 1e-3),
                 "max_rel_diff_from_labelled_sum": float(((Sm - ref).abs() / ref.abs().clamp_min(1e-300)).max()),
                 "states_per_config": B.plan_counts_mask_only(nn, True)["states"]}
    cdet = cdet_comparison(B, torch, G, S, n.size, nn, w.nflav, stream)
    return {"workload": "honeycomb: 16x16 cells, beta=5, SU(2) flavour-dependent (staggered field +-0.3), "
                        "mu=0.3, n=8, %d configs, sublattice labels summed (2n x 2n matrices)" % n.size,
            "configs_per_s": n.size / (ms * 1e-3), "ms_per_batch_incl_g0": ms, "forward_levels_ms": fwd_ms,
            "kernel": "sub_fwd_kernel<8, true, false>", "launch_shape": shape,
            "flop_per_config": flop, "forward_tflops": flop * n.size / (fwd_ms * 1e-3) / 1e12,
            "frac_of_fp64_peak": flop * n.size / (fwd_ms * 1e-3) / PEAK_FP64,
            "state_stream_bytes_per_config": states_bytes,
            "state_stream_TBps": states_bytes * n.size / (fwd_ms * 1e-3) / 1e12,
            "gradient_step": grad,
            "mask_only_alg1": mask_only,
            "cdet_comparison": cdet}


def mask_only_su2(B, torch, reps):
    """The mask-only variant (Alg. 1) against the vertex-level two-flavour path
    on the same SU(2) propagators: the adjoint workload's configurations
    (8x8, beta=4, n=10, 2048) with mu=-0.5 for both spins; forward + reverse
    sweep each, autotuned; the two sums agree up to the factor 2^n."""
    from paper_2507_12349_amd.autograd import Geometry
    from paper_2507_12349_amd.workloads import draw
    d = draw(WORKLOAD)
    w = d.workload
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    nconf, n = int(d.n.size), int(d.n[0])
    geo = Geometry(d, 2, dev)
    G = torch.empty(geo.total, dtype=torch.float64, device=dev)
    dG = torch.empty_like(G)
    B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, np.array([w.mu[0]] * 2),
               np.zeros(2), geo.Goff, G, dG, stream)
    ob = torch.ones(nconf, dtype=torch.float64, device=dev)
    res = {}
    outs = {}
    for name, mask in (("mask_only", True), ("vertex_two_flavour", False)):
        b = B.Batch(d.n, 2, B.FLAVOUR, mask_only=mask)
        S = torch.empty(nconf, dtype=torch.float64, device=dev)
        Gb = torch.empty_like(G)
        b.autotune(G, geo.Goff, None, -1.0, S, ob, Gb, None, stream=stream)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        f0, f1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        f0.record(stream)
        for _ in range(reps):
            b.forward(G, geo.Goff, None, -1.0, S, stream)
        f1.record(stream)
        e0.record(stream)
        for _ in range(reps):
            b.adjoint(G, geo.Goff, None, -1.0, ob, S, Gb, None, stream)
        e1.record(stream)
        torch.cuda.synchronize()
        outs[name] = S.clone() / (1.0 if mask else float(2 ** n))
        res[name] = {"forward_configs_per_s": nconf / (f0.elapsed_time(f1) / reps * 1e-3),
                     "fwd_adjoint_configs_per_s": nconf / (e0.elapsed_time(e1) / reps * 1e-3),
                     "launch_shape": b.launch_shape(n)}
        b.close()
    pm, pv = B.plan_counts_mask_only(n), B.plan_counts(n)
    res["states_per_config"] = {"mask_only": pm["states"], "vertex_two_flavour": 2 * pv["states"]}
    res["extensions_per_config"] = {"mask_only": pm["ext"], "vertex_two_flavour": 2 * pv["ext"]}
    a, v = outs["mask_only"], outs["vertex_two_flavour"]
    res["max_rel_diff_of_sums"] = float(((a - v).abs() / v.abs().clamp_min(1e-300)).max())
    res["workload"] = ("adjoint workload's configurations as SU(2): 8x8, beta=4, mu=-0.5 both spins, n=%d, "
                       "%d configs; the vertex-level sum divided by 2^n" % (n, nconf))
    return res


def cdet_comparison(B, torch, G, S, nconf, n, nflav, stream):
    """The CDet path (3^n labelled principal minors with pseudo-pivots, then
    the connected recursion) on the honeycomb propagators the labelled DP just
    summed, in FP64 and in double-double: rate, and deviation from the DP
    (whose sum over the 2^n label assignments equals 2^n times CDet's)."""
    assert nflav == 2
    A = G.reshape(nconf, 2, 2 * n, 2 * n)
    cos = S / float(2 ** n)
    res = {}
    for prec, name in ((0, "fp64"), (1, "double_double")):
        out = torch.empty(nconf, dtype=torch.float64, device=G.device)
        B.cdet_su2(A, n, prec, out, 1e-12, stream)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        B.cdet_su2(A, n, prec, out, 1e-12, stream)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1)
        rel = ((out - cos).abs() / cos.abs().clamp_min(1e-300)).cpu().numpy()
        res[name] = {"configs_per_s": nconf / (ms * 1e-3), "ms_per_batch": ms,
                     "rel_dev_from_dp_median": float(np.median(rel)), "rel_dev_from_dp_max": float(np.max(rel))}
    return res


def mc_series(torch, orders=8, nconf=8192, nbatches=4):
    """Monte Carlo series of the interaction correction to ln Z per site and
    unit time on the adjoint workload's lattice (8x8, beta=4, mu=-0.5, SU(4),
    U=1) through the device driver, and its Pade band ([m/m], m = 1..4, at
    xi = 1).  Reports the sampling rate at the highest order."""
    from paper_2507_12349_amd import mc
    kw = dict(L=8, t=1.0, beta=4.0, mu=[-0.5], alpha=[0.0], nflav=4, variant=0, U=1.0, nconf=nconf,
              nbatches=nbatches)
    coefs, top_ms = [], None
    for n in range(1, orders + 1):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        c = mc.lnz_coefficient(n, seed=2024 + n, **kw)
        e1.record()
        torch.cuda.synchronize()
        coefs.append(c)
        top_ms = e0.elapsed_time(e1)
    a = np.array([0.0] + [c.value for c in coefs])
    da = np.array([0.0] + [c.error for c in coefs])
    degrees = [m for m in (1, 2, 3, 4) if 2 * m <= orders]
    try:
        lo, hi, vals, errs = mc.pade_band(a, da, degrees)
        pade = {"degrees": degrees, "values": vals, "errors": errs, "band": [lo, hi]}
    except Exception as exc:   # an approximant may not exist for a given series
        pade = {"error": str(exc)}
    return {"workload": "8x8 square lattice, beta=4, mu=-0.5, SU(4) uniform, U=1; vertex 0 fixed, %d x %d "
                        "samples per order" % (nbatches, nconf),
            "coefficients": [{"n": c.n, "value": c.value, "error": c.error} for c in coefs],
            "samples_per_s_at_top_order": nconf * nbatches / (top_ms * 1e-3),
            "pade_of_correction_at_xi_1": pade}


def _flop_per_config(B, n, nflav, variant, stubs):
    """Algorithmic FLOP of one forward sum (2 per FMA): every extension and
    close transition once per flavour slot, plus the shift-head transitions."""
    pc = B.plan_counts(int(n))
    nfs = nflav if variant == 1 else 1
    return 2.0 * nfs * (pc["ext"] + pc["closes"]) + (2.0 * nfs * pc["stub_edges"] if stubs else 0.0)


def _refs_stats(name, S_host, idx_all=None):
    """Deviation of sums computed on the GPU's own propagators from the
    oracle's references (tests/golden/refs_NAME.npz, long double DP on the
    oracle's propagators; the two propagator builds differ in the last bits,
    so this is a consistency figure, not the parity gate of the tests) and the
    cancellation kappa = S_abs / |S| of the referenced configurations."""
    path = os.path.join(ROOT, "tests", "golden", "refs_%s.npz" % name)
    if not os.path.exists(path):
        return None
    r = np.load(path)
    idx = r["idx"]
    rel = np.abs(S_host[idx] - r["S"]) / np.abs(r["S"])
    kappa = r["S_abs"] / np.abs(r["S"])
    low = kappa <= 1e5
    return {"configs": int(idx.size), "rel_dev_median": float(np.median(rel)),
            "rel_dev_max_kappa_le_1e5": float(rel[low].max()) if low.any() else None,
            "rel_dev_max": float(rel.max()),
            "kappa_median": float(np.median(kappa)), "kappa_p90": float(np.quantile(kappa, 0.9)),
            "kappa_max": float(kappa.max()), "configs_kappa_gt_1e5": int((~low).sum())}


def _cpu_forward_rate(d, idx, threads, variant, nflav, stubs_of, per_config=None):
    """Oracle DP (float64) forward sums of configurations idx, one per thread:
    configurations per second and wall time.  per_config, a dict, receives each
    configuration's own time on its thread."""
    from concurrent.futures import ThreadPoolExecutor

    import oracle
    from oracle import g0
    w = d.workload
    oracle.build(force=False)
    mats = {}
    for c in idx:
        sites, tau = d.config(c)
        nmat = nflav if variant == 1 else 1
        alpha = np.asarray(d.delta[:nmat]) if variant == 1 else np.zeros(1)
        G, _ = g0.build_g0(w.L, w.t, w.beta, np.asarray(w.mu[:nmat]), alpha, sites, tau)
        mats[c] = G[0] if variant == 0 else G

    def one(c):
        t = time.perf_counter()
        r = oracle.dp(mats[c], nflav, variant, stubs_of(c), -1.0, precision="d")
        if per_config is not None:
            per_config[c] = time.perf_counter() - t
        return r

    t0 = time.perf_counter()
    with ThreadPoolExecutor(max_workers=threads) as ex:
        list(ex.map(one, idx))
    dt = time.perf_counter() - t0
    return len(idx) / dt, dt


def workload_legs(B, torch, reps, cpu_threads=0, only=None):
    """The other workloads of the measurement plan, forward sums on the GPU
    with inputs resident (propagator kernel + batched levels), autotuned:
      plain_single  (4x4, beta=2, SU(2), n=4, 1 config): plain call latency
      plain_batch   (8x8, beta=4, SU(4), n=8, 4096): batched vs one call per config
      sym_broken    (8x8, beta=4, SU(3) flavour mu, n=10, 1024)
      uneven        (16x16, beta=5, SU(6) shifts, n=6..12, 8192): graph replay
    each with configs/s, algorithmic FP64 TFLOP/s against the 78.6 TFLOP/s
    peak, the deviation from the oracle's references and their kappa; with
    cpu_threads the oracle's forward on a small sample beside it."""
    from paper_2507_12349_amd.autograd import Geometry
    from paper_2507_12349_amd.workloads import draw
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    out = {}

    def ev():
        return torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    for name in ("plain_single", "plain_batch", "sym_broken", "uneven"):
        if only and name != only:
            continue
        d = draw(name)
        w = d.workload
        nmat = w.nflav if w.variant == 1 else 1
        mu = np.asarray(w.mu[:nmat])
        alpha = np.asarray(d.delta[:nmat]) if w.variant == 1 else np.zeros(1)
        geo = Geometry(d, nmat, dev)
        nconf = geo.nconf
        G = torch.empty(geo.total, dtype=torch.float64, device=dev)
        st = None
        if w.stubs:
            st = torch.as_tensor(np.tile(d.delta[:nmat] / w.U, (nconf, 1)), device=dev)
        b = B.Batch(d.n, w.nflav, w.variant, stubs=st is not None)
        S = torch.empty(nconf, dtype=torch.float64, device=dev)

        def g0(s=stream):
            B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, mu, alpha, geo.Goff, G, None, s)

        g0()
        b.autotune(G, geo.Goff, st, -1.0, S, stream=stream)
        fpc = {int(k): _flop_per_config(B, k, w.nflav, w.variant, st is not None) for k in np.unique(d.n)}
        flop = float(sum(fpc[int(k)] * int((d.n == k).sum()) for k in fpc))
        leg = {"workload": w.note, "nconf": nconf}
        if name == "uneven":
            # the whole step (propagators + every order's level launches) replayed from one graph
            cs = torch.cuda.Stream()
            cs.wait_stream(stream)
            with torch.cuda.stream(cs):
                g0(cs)
                b.forward(G, geo.Goff, st, -1.0, S, cs)
            stream.wait_stream(cs)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=cs):
                g0(cs)
                b.forward(G, geo.Goff, st, -1.0, S, cs)
            graph.replay()
            torch.cuda.synchronize()
            e0, e1 = ev()
            e0.record(stream)
            for _ in range(reps):
                graph.replay()
            e1.record(stream)
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / reps
            leg["graph_replay"] = True
            leg["orders"] = {int(k): int((d.n == k).sum()) for k in np.unique(d.n)}
        else:
            g0()
            b.forward(G, geo.Goff, st, -1.0, S, stream)
            torch.cuda.synchronize()
            e0, e1 = ev()
            e0.record(stream)
            for _ in range(reps):
                g0()
                b.forward(G, geo.Goff, st, -1.0, S, stream)
            e1.record(stream)
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / reps
        # the level launches alone (phase events on the launch stream)
        b.timing(True)
        for _ in range(reps):
            b.forward(G, geo.Goff, st, -1.0, S, stream)
        ph, _ = b.timing_read()
        b.timing(False)
        lv_ms = ph["forward"] / reps
        leg.update({"configs_per_s": nconf / (ms * 1e-3), "ms_per_batch_incl_g0": ms, "forward_levels_ms": lv_ms,
                    "flop_per_config_mean": flop / nconf, "forward_tflops": flop / (lv_ms * 1e-3) / 1e12,
                    "frac_of_fp64_peak": flop / (lv_ms * 1e-3) / PEAK_FP64,
                    "launch_shapes": {int(k): b.launch_shape(int(k)) for k in np.unique(d.n)}})
        S_host = S.cpu().numpy()
        if name in ("plain_batch", "sym_broken"):
            # forward + reverse sweep (the adjoint call, reverse launch shapes autotuned too)
            ob = torch.ones(nconf, dtype=torch.float64, device=dev)
            Gb = torch.empty_like(G)
            sb = None if st is None else torch.empty_like(st)
            Sa = torch.empty_like(S)
            b.autotune(G, geo.Goff, st, -1.0, Sa, ob, Gb, sb, stream=stream)
            b.adjoint(G, geo.Goff, st, -1.0, ob, Sa, Gb, sb, stream)
            torch.cuda.synchronize()
            a0, a1 = ev()
            a0.record(stream)
            for _ in range(reps):
                b.adjoint(G, geo.Goff, st, -1.0, ob, Sa, Gb, sb, stream)
            a1.record(stream)
            torch.cuda.synchronize()
            ams = a0.elapsed_time(a1) / reps
            leg.update({"fwd_adjoint_configs_per_s": nconf / (ams * 1e-3), "fwd_adjoint_ms": ams,
                        "adjoint_S_equals_forward": bool(torch.equal(Sa, S))})
            del Gb, sb, Sa
        if name in ("plain_single", "plain_batch"):
            # the plain form: one call per configuration (a launch per level, one of 64 lanes busy)
            n0 = int(d.n[0])
            one = B.Batch([n0], w.nflav, w.variant)
            Sp = torch.empty_like(S)
            nn = nmat * n0 * n0
            goff = geo.Goff_host
            for c in range(min(nconf, 16)):
                one.forward(G[int(goff[c]):int(goff[c]) + nn], None, None, -1.0, Sp[c:c + 1], stream)
            torch.cuda.synchronize()
            npl = nconf if nconf > 1 else 200
            p0, p1 = ev()
            p0.record(stream)
            for i in range(npl):
                c = i % nconf
                one.forward(G[int(goff[c]):int(goff[c]) + nn], None, None, -1.0, Sp[c:c + 1], stream)
            p1.record(stream)
            torch.cuda.synchronize()
            one.close()
            plain = npl / (p0.elapsed_time(p1) * 1e-3)
            leg.update({"plain_configs_per_s": plain, "batched_over_plain": leg["configs_per_s"] / plain,
                        "plain_equals_batched_bitwise": bool(torch.equal(Sp, S)),
                        "plain_note": "one call per configuration: %s, with one of the 64 lanes of each wavefront busy"
                                      % ("a launch per level" if n0 > 5 else "the levels in one launch")})
            if name == "plain_single":
                Gh = G.cpu().numpy().reshape(nmat, n0, n0)
                t0 = time.perf_counter()
                for _ in range(50):
                    B.connected_sum_host(Gh[0] if w.variant == 0 else Gh, w.nflav, w.variant)
                leg["host_call_configs_per_s"] = 50 / (time.perf_counter() - t0)
        leg["vs_oracle_refs"] = _refs_stats(name, S_host)
        if cpu_threads:
            if name == "uneven":
                # a seeded subsample per order (the batch's first configurations of that
                # order), timed configuration by configuration on all cores, largest orders
                # first; the per-order mean single-thread time is extrapolated to the batch's
                # order mix.  64 per order up to n = 10; fewer at n = 11, 12 (5 and 19 s each)
                # so that the run stays within about half a minute.
                take = {k: (64 if k <= 10 else 32 if k == 11 else 8) for k in range(6, 13)}
                idx = []
                for k in range(12, 5, -1):
                    idx += [int(c) for c in np.nonzero(d.n == k)[0][:take[k]]]
                sig = d.delta[:nmat] / w.U
                tc = {}
                _, wall = _cpu_forward_rate(d, idx, cpu_threads, w.variant, w.nflav, lambda c: sig,
                                            per_config=tc)
                tk = {k: float(np.mean([tc[c] for c in idx if int(d.n[c]) == k])) for k in range(6, 13)}
                core_s = sum(tk[k] * int((d.n == k).sum()) for k in tk)
                leg["cpu_oracle"] = {"configs_per_s": nconf / (core_s / cpu_threads), "cores": cpu_threads,
                                     "kind": "oracle, extrapolated",
                                     "sample": "%s configurations of orders 6..12 (%d in all, %.0f s wall on %d "
                                               "threads); mean time per configuration and order x the batch's "
                                               "order counts / %d cores"
                                               % ("/".join(str(take[k]) for k in range(6, 13)), len(idx), wall,
                                                  cpu_threads, cpu_threads),
                                     "configs_per_order_timed": {int(k): take[k] for k in range(6, 13)},
                                     "s_per_config_per_order": {int(k): v for k, v in tk.items()}}
            else:
                k = {"plain_single": 1, "plain_batch": 256, "sym_broken": 48}[name]
                rate, dt = _cpu_forward_rate(d, list(range(k)), cpu_threads, w.variant, w.nflav, lambda c: None)
                leg["cpu_oracle"] = {"configs_per_s": rate, "cores": cpu_threads, "kind": "oracle",
                                     "sample": "first %d configurations, float64 DP forward, %.1f s wall" % (k, dt)}
        b.close()
        out[name] = leg
        del G, S
    return out


def cpu_baseline(d, nsample, threads):
    """The oracle (C, float64) on host cores: propagators (numpy), reverse sweep
    with the forward sum (oracle DP), chain rule; one configuration per task."""
    from concurrent.futures import ThreadPoolExecutor

    import oracle
    from oracle import g0
    w = d.workload
    oracle.build(force=False)

    def one(c):
        sites, tau = d.config(c)
        G, dG = g0.build_g0(w.L, w.t, w.beta, np.array(w.mu[:1]), np.zeros(1), sites, tau)
        S, Gb, sb = oracle.dp_adjoint(G[0], w.nflav, 0, np.zeros(1), precision="d")
        xb = float(np.sum(Gb * dG[0]))
        return S, -xb, (xb + sb[0] / w.U) / w.nflav

    one(0)
    t0 = time.perf_counter()
    with ThreadPoolExecutor(max_workers=threads) as ex:
        list(ex.map(one, range(nsample)))
    dt = time.perf_counter() - t0
    return nsample / dt, dt


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--nconf", type=int, default=0)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-tune", action="store_true", help="default launch shapes instead of autotuned ones")
    ap.add_argument("--no-honeycomb", action="store_true", help="skip the sublattice (honeycomb) measurement")
    ap.add_argument("--no-mc", action="store_true", help="skip the Monte Carlo series measurement")
    ap.add_argument("--no-mask-only", action="store_true", help="skip the SU(2) mask-only comparison")
    ap.add_argument("--no-workloads", action="store_true",
                    help="skip the other workloads (plain single, plain batch, symmetry broken, uneven)")
    ap.add_argument("--cpu-sample", type=int, default=1536)
    ap.add_argument("--leg", choices=("plain_single", "plain_batch", "sym_broken", "uneven", "honeycomb"),
                    help="run only this workload's leg (for profiling; with --counters after the calibration copy)")
    ap.add_argument("--counters", action="store_true",
                    help="run one calibration copy (1 GiB), one batched forward and one adjoint, "
                         "then exit (for rocprofv3 --pmc passes)")
    ap.add_argument("--shape", default=None,
                    help="with --counters: launch shape FWD_WAVES,FWD_MASKS,ADJ_MASKS of the adjoint workload's "
                         "calls (the autotuner's choice of a timed run; default: the library's default shape)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the configurations are independent and a "
              "multi-GPU run would shard them with no collective on the hot path; run with --gpus 1.",
              file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2507_12349_amd import _binding as B
    from paper_2507_12349_amd.autograd import Geometry
    from paper_2507_12349_amd.workloads import draw

    if args.leg:
        if args.counters:
            src = torch.ones(1 << 27, dtype=torch.float64, device="cuda:0")
            torch.empty_like(src).copy_(src)
            torch.cuda.synchronize()
            del src
        reps = 1 if args.counters else max(3, args.steps // 2)
        if args.leg == "honeycomb":
            res = honeycomb_forward(B, torch, reps)
        else:
            res = workload_legs(B, torch, reps, 0, only=args.leg)[args.leg]
        print(json.dumps({"leg": args.leg, "result": res}), flush=True)
        return

    d = draw(WORKLOAD, nconf=args.nconf or None)
    w = d.workload
    nconf = int(d.n.size)
    n = int(d.n[0])
    dev = torch.device("cuda:0")
    geo = Geometry(d, 1, dev)
    mu, alpha = np.array(w.mu[:1]), np.zeros(1)
    G = torch.empty(geo.total, dtype=torch.float64, device=dev)
    dG = torch.empty_like(G)
    Gb = torch.empty_like(G)
    stub = torch.zeros((nconf, 1), dtype=torch.float64, device=dev)
    sb = torch.empty_like(stub)
    S = torch.empty(nconf, dtype=torch.float64, device=dev)
    obar = torch.ones(nconf, dtype=torch.float64, device=dev)
    mub = torch.empty(nconf, dtype=torch.float64, device=dev)
    alb = torch.empty(nconf, dtype=torch.float64, device=dev)
    batch = B.Batch(d.n, w.nflav, 0, stubs=True)
    fwd_batch = B.Batch(d.n, w.nflav, 0, stubs=False)
    stream = torch.cuda.current_stream()

    if args.counters:
        # a plain copy of known size calibrates the HBM byte counters
        src = torch.ones(1 << 27, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        if args.shape:
            fw, fm, am = (int(x) for x in args.shape.split(","))
            fwd_batch.set_launch_shape(n, fw, fm, am)
            batch.set_launch_shape(n, fw, fm, am)
        B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, mu, alpha, geo.Goff, G, dG, stream)
        fwd_batch.forward(G, geo.Goff, None, -1.0, S, stream)
        batch.adjoint(G, geo.Goff, stub, -1.0, obar, S, Gb, sb, stream)
        torch.cuda.synchronize()
        if not args.no_honeycomb:
            honeycomb_forward(B, torch, 1)
            torch.cuda.synchronize()
        print(json.dumps({"counters_pass": "done", "copy_bytes": 2 * 8 * (1 << 27)}), flush=True)
        return

    # launch shapes: autotuned once on the batch's own inputs (untimed set-up)
    if not args.no_tune:
        B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, mu, alpha, geo.Goff, G, dG, stream)
        fwd_batch.autotune(G, geo.Goff, None, -1.0, S, stream=stream)
        batch.autotune(G, geo.Goff, stub, -1.0, S, obar, Gb, sb, stream=stream)
    shape = batch.launch_shape(n)

    def evpair():
        return torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def step(e=None, st=stream):
        if e: e["g0"][0].record(st)
        B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, mu, alpha, geo.Goff, G, dG, st)
        if e: e["g0"][1].record(st); e["adj"][0].record(st)
        batch.adjoint(G, geo.Goff, stub, -1.0, obar, S, Gb, sb, st)
        if e: e["adj"][1].record(st); e["chain"][0].record(st)
        B.chain_mu_shift(nconf, geo.n, 1, geo.Goff, Gb, dG, sb, 1, w.U, mub, alb, st)
        if e: e["chain"][1].record(st)

    for _ in range(args.warmup):
        step()
    # per-step events (read after the timed region) and the library's phase
    # events, all on the stream the kernels run on
    evs = [{k: evpair() for k in ("g0", "adj", "chain")} for _ in range(args.steps)]
    batch.timing(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        step(evs[i])
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    phases, ncalls = batch.timing_read()
    batch.timing(False)
    assert ncalls == args.steps
    acc = {k: sum(e[k][0].elapsed_time(e[k][1]) for e in evs) for k in ("g0", "adj", "chain")}
    ms_step = 1e3 * wall / args.steps
    value = nconf / (wall / args.steps)

    # the same step replayed from a HIP graph (captured once; no host launches)
    graph = torch.cuda.CUDAGraph()
    cs = torch.cuda.Stream()
    cs.wait_stream(stream)
    with torch.cuda.stream(cs):
        step(st=cs)
    stream.wait_stream(cs)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=cs):
        step(st=cs)
    graph.replay()
    torch.cuda.synchronize()
    ge0, ge1 = evpair()
    ge0.record(stream)
    for _ in range(args.steps):
        graph.replay()
    ge1.record(stream)
    torch.cuda.synchronize()
    graph_ms = ge0.elapsed_time(ge1) / args.steps

    # batched forward alone (G0 + forward) and the plain one-launch-per-config form
    def fwd_batched():
        B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, mu, alpha, geo.Goff, G, dG, stream)
        fwd_batch.forward(G, geo.Goff, None, -1.0, S, stream)

    for _ in range(3):
        fwd_batched()
    torch.cuda.synchronize()
    fe0, fe1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    fk0, fk1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    reps = max(3, args.steps // 2)
    fwd_kernel_ms = 0.0
    fe0.record(stream)
    for _ in range(reps):
        B.build_g0(nconf, geo.n, geo.voff, geo.sites, geo.tau, w.L, w.t, w.beta, mu, alpha, geo.Goff, G, dG, stream)
        fk0.record(stream)
        fwd_batch.forward(G, geo.Goff, None, -1.0, S, stream)
        fk1.record(stream)
        fk1.synchronize()
        fwd_kernel_ms += fk0.elapsed_time(fk1)
    fe1.record(stream)
    torch.cuda.synchronize()
    fwd_ms = fe0.elapsed_time(fe1) / reps
    fwd_kernel_ms /= reps
    S_batched = S.clone()

    one = B.Batch([n], w.nflav, 0, stubs=False)
    Sp = torch.empty_like(S)
    nn = n * n
    goff = geo.Goff_host
    for c in range(min(nconf, 32)):
        one.forward(G[int(goff[c]):int(goff[c]) + nn], None, None, -1.0, Sp[c:c + 1], stream)
    torch.cuda.synchronize()
    pe0, pe1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    pe0.record(stream)
    for c in range(nconf):
        one.forward(G[int(goff[c]):int(goff[c]) + nn], None, None, -1.0, Sp[c:c + 1], stream)
    pe1.record(stream)
    torch.cuda.synchronize()
    plain_ms = pe0.elapsed_time(pe1)
    plain_equal = bool(torch.equal(Sp, S_batched))
    # the plain form synchronised after every configuration (host round trip per call)
    nsync = min(nconf, 256)
    t0s = time.perf_counter()
    for c in range(nsync):
        one.forward(G[int(goff[c]):int(goff[c]) + nn], None, None, -1.0, Sp[c:c + 1], stream)
        stream.synchronize()
    plain_sync_rate = nsync / (time.perf_counter() - t0s)
    one.close()

    # the plain form of the adjoint call (forward recomputed + reverse sweep),
    # one configuration per call, on the first configurations of the batch
    one_adj = B.Batch([n], w.nflav, 0, stubs=True)
    nadj = min(nconf, 256)
    Sa = torch.empty(nadj, dtype=torch.float64, device=dev)
    Gba = torch.empty(nadj * nn, dtype=torch.float64, device=dev)
    sba = torch.empty((nadj, 1), dtype=torch.float64, device=dev)

    def adj_plain(c):
        a0 = int(goff[c])
        one_adj.adjoint(G[a0:a0 + nn], None, stub[c:c + 1], -1.0, obar[c:c + 1], Sa[c:c + 1],
                        Gba[c * nn:(c + 1) * nn], sba[c:c + 1], stream)

    for c in range(min(nadj, 8)):
        adj_plain(c)
    torch.cuda.synchronize()
    ae0, ae1 = evpair()
    ae0.record(stream)
    for c in range(nadj):
        adj_plain(c)
    ae1.record(stream)
    torch.cuda.synchronize()
    adj_plain_rate = nadj / (ae0.elapsed_time(ae1) * 1e-3)
    one_adj.close()
    # reference: the batched adjoint call on the same inputs
    batch.adjoint(G, geo.Goff, stub, -1.0, obar, S, Gb, sb, stream)
    torch.cuda.synchronize()
    adj_plain_S_equal = bool(torch.equal(Sa, S[:nadj]))
    gref = Gb[:nadj * nn]
    adj_plain_grad_dev = float(((Gba - gref).abs().max() / gref.abs().max()).item())

    # the same adjoint call with deterministic gradients (fixed summation order)
    det_batch = B.Batch(d.n, w.nflav, 0, stubs=True, deterministic=True)
    Gbd, sbd = torch.empty_like(Gb), torch.empty_like(sb)
    det_batch.adjoint(G, geo.Goff, stub, -1.0, obar, S, Gbd, sbd, stream)
    torch.cuda.synchronize()
    de0, de1 = evpair()
    de0.record(stream)
    for _ in range(reps):
        det_batch.adjoint(G, geo.Goff, stub, -1.0, obar, S, Gbd, sbd, stream)
    de1.record(stream)
    torch.cuda.synchronize()
    det_ms = de0.elapsed_time(de1) / reps
    Gbd2 = torch.empty_like(Gb)
    det_batch.adjoint(G, geo.Goff, stub, -1.0, obar, S, Gbd2, sbd, stream)
    torch.cuda.synchronize()
    deterministic = {"adjoint_call_ms": det_ms, "adjoint_configs_per_s": nconf / (det_ms * 1e-3),
                     "slowdown_vs_default_adjoint": det_ms / (acc["adj"] / args.steps),
                     "repeat_bitwise_equal": bool(torch.equal(Gbd, Gbd2)),
                     "max_dev_from_default_rel_to_max": float(((Gbd - Gb).abs().max() / Gb.abs().max()).item())}
    det_batch.close()
    del Gbd, Gbd2, sbd

    # roofline of the dominant kernel, the reverse level kernel: one launch
    # per level, 2n - 2 launches per sweep (one vertex's two visits stay inside
    # the launches); algorithmic FLOP of the sweep per
    # configuration = 4 (E + C) (the adjoint of every extension and close
    # edge: one FMA into B, one into dS/dG)
    pc = B.plan_counts(n)
    flop_fwd = 2.0 * (pc["ext"] + pc["closes"])
    flop_rev = 2.0 * flop_fwd
    nlaunch = 2 * n - 2
    rev_ms = phases["reverse"] / args.steps            # per sweep
    launch_ms = rev_ms / nlaunch                       # average launch
    flop_launch = flop_rev * nconf / nlaunch
    achieved = flop_launch / (launch_ms * 1e-3)
    rev_kernel = REV_KERNEL % n
    traffic = _traffic(rev_kernel)
    hbm = None
    if traffic is not None:
        ai = flop_launch / traffic
        hbm = {"bytes_per_launch": traffic, "achieved_GBps": traffic / (launch_ms * 1e-3) / 1e9,
               "frac_of_8TBps": traffic / (launch_ms * 1e-3) / PEAK_HBM,
               "ai_flop_per_byte": ai,
               "frac_of_attainable": achieved / min(PEAK_FP64, ai * PEAK_HBM)}

    hc = None if args.no_honeycomb else honeycomb_forward(B, torch, max(3, args.steps // 2))
    mcs = None if args.no_mc else mc_series(torch)
    mo = None if args.no_mask_only else mask_only_su2(B, torch, max(3, args.steps // 2))

    nproc = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    # the host share of one GPU on the measurement boxes is 16 cores
    threads = max(1, min(16, nproc))
    S_host = S.cpu().numpy()
    legs = None if args.no_workloads else workload_legs(B, torch, max(3, args.steps // 2),
                                                        0 if args.no_cpu else threads)
    cpu = None
    if not args.no_cpu:
        rate, dt = cpu_baseline(d, args.cpu_sample, threads)
        rate1, dt1 = cpu_baseline(d, 16, 1)
        cpu = {"value": rate, "unit": "configs/s", "cores": threads, "kind": "oracle",
               "sample": "%d configs of the same workload (propagators, float64 DP forward + reverse sweep, "
                         "chain rule), one config per thread, %.1f s wall" % (args.cpu_sample, dt),
               "host_cpus_visible": nproc,
               "single_core_value": rate1,
               "single_core_sample": "16 configs on one thread, %.1f s" % dt1}

    rec = {
        "metric": "connected-sum configs/sec at n=10 SU(4) FP64 (batched vs plain; fwd+adjoint)",
        "value": value,
        "unit": "configs/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic (seeded uniform sites and times, 8x8 lattice)",
        "config": {"workload": "adjoint: 8x8 lattice, beta=4, mu=-0.5, SU(4) uniform, n=10, "
                               "%d configs, forward + reverse sweep + chain rule to mu and shift" % nconf,
                   "n": n, "nflav": w.nflav, "nconf": nconf,
                   "parallelism": "single GPU; 64 configurations per wavefront, one launch per DP level",
                   "launch_shape": shape, "autotuned": not args.no_tune},
        "breakdown_ms": {"g0": acc["g0"] / args.steps, "adjoint_incl_forward": acc["adj"] / args.steps,
                         "chain": acc["chain"] / args.steps,
                         "adjoint_phases": {k: v / args.steps for k, v in phases.items()}},
        "graph_replay": {"ms_per_step": graph_ms, "configs_per_s": nconf / (graph_ms * 1e-3)},
        "forward_batched_configs_per_s": nconf / (fwd_ms * 1e-3),
        "forward_kernel_ms": fwd_kernel_ms,
        "forward_plain_configs_per_s": nconf / (plain_ms * 1e-3),
        "forward_plain_synced_configs_per_s": plain_sync_rate,
        "plain_note": "one call per configuration: a launch per level with one of the 64 lanes of each wavefront busy",
        "batched_over_plain": (nconf / (fwd_ms * 1e-3)) / (nconf / (plain_ms * 1e-3)),
        "plain_equals_batched_bitwise": plain_equal,
        "adjoint_batched_configs_per_s": nconf / (acc["adj"] / args.steps * 1e-3),
        "adjoint_plain_configs_per_s": adj_plain_rate,
        "adjoint_batched_over_plain": (nconf / (acc["adj"] / args.steps * 1e-3)) / adj_plain_rate,
        "adjoint_plain_check": {"configs": nadj, "S_equals_batched_bitwise": adj_plain_S_equal,
                                "max_grad_dev_rel_to_max": adj_plain_grad_dev},
        "deterministic_gradients": deterministic,
        "vs_oracle_refs": _refs_stats(WORKLOAD, S_host) if nconf == 2048 else None,
        "roofline": {"bound": "alu", "kernel": rev_kernel,
                     "note": "bound = the method's: FP64 ALU on algorithmic FLOP; the kernel itself streams every "
                             "DP state through HBM (see hbm: AI ~1 FLOP/B, below the 9.8 FLOP/B ridge), which caps "
                             "frac near AI x 8 TB/s / 78.6 TFLOP/s",
                     "unit_of_work": "one launch = one level of the reverse sweep over all %d configs "
                                     "(%d launches per sweep; per-launch figures are sweep averages)" % (nconf, nlaunch),
                     "achieved": achieved / 1e12, "peak": PEAK_FP64 / 1e12, "unit": "TFLOP/s",
                     "frac": achieved / PEAK_FP64, "traffic": traffic,
                     "flop_per_launch": flop_launch, "avg_launch_ms": launch_ms,
                     "flop_per_config_sweep": flop_rev, "hbm": hbm,
                     "forward_kernel_tflops": flop_fwd * nconf / (phases["forward"] / args.steps * 1e-3) / 1e12},
        "workloads": legs,
        "sublattice_honeycomb_forward": hc,
        "mc_series": mcs,
        "su2_mask_only_vs_vertex": mo,
        "cpu_baseline": cpu,
    }
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
