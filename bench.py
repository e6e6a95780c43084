"""Benchmark of the differentiable propagation hot path on one MI355X.

One step = one pass of the whole path over one batch of synthetic input:
build the system (single-mode builders, FP64 eigensolves, FP64 stage tables),
propagate all columns with the fused RK4 (checkpoints kept), reduce the
fidelity and seed the costate, run the adjoint and assemble the gradient.

Workload: the 8-transmon ring (d=3, D=6561), 256 computational columns,
T=60 ns, 3000 RK4 steps, 40 parameters.  Metric: RK4 steps * dim^2 / s,
read as sum over solves of N * D * S per second (S = number of propagated
columns).  Parity on the same run, in the same launch configuration (all 256
columns): the composite state cost (Sec. 4.1) of the 8 seeded sampled columns
against stored targets near the oracle's own final states (F ~ 0.99) and its
gradient, against the stored CPU FP64 oracle result; and the CZ target
restricted to the sampled computational states (F ~ 5e-7).

The timed steps evaluate the generator with the rotated complex operators
(``--frame complex``, the default): their gradient meets the 1e-4 bar on the
F ~ 0.99 target.  The real frame (real operators between diagonal frame
rotations) is faster but its FP32 gradient there is ~2e-4; the line reports its
time and parity beside the timed evaluation (``ms_per_step_real_frame``,
``grad_rel_err_real_frame``), or the reverse with ``--frame real``.

The roofline object is that of the dominant kernel, the adjoint's reverse
kernel (about 60 % of a step); the forward and the recompute kernels follow in
``kernels``.  Kernel durations come from HIP events the library records on the
launch stream around every launch (scp_system_set_timing).

Beside the timed steps (not part of ``value``): one forward of the same
workload on the plain complex FP64 GPU path (the speedup denominator), the
open-system (Lindblad) propagation of a 4-fluxonium chain's 256 computational
matrix units (``open_system``), the second-order product formula on the
4-fluxonium chain with its LCAM gradient (``product_formula``), and a serving replay of the first requests of the mixed request stream (2-6 modes,
d in {3,4,5}, T in [20,200] ns, half with gradients): saturated throughput,
then Poisson arrivals at 0.5x and 0.9x that throughput, with p50/p99 latency.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline]
                    [--serve-requests R] [--no-plain64] [--no-lindblad]
                    [--no-product-formula]
    python bench.py --lindblad | --trotter | --configs | --cpu-protocol
"""
from __future__ import annotations

import argparse
import glob
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP32 = 157.3e12      # MI355X FP32 (vector incl. packed, and dense MFMA), FLOP/s
PEAK_HBM = 8.0e12         # bytes/s


def contraction_counts(desc):
    """(C_fwd per generator application, sensitivity passes per adjoint stage)."""
    pairs = set()
    first = set()
    for c in desc["couplings"]:
        pairs.add(((c["i"], c["op_i"]), c["j"]))
        first.add((c["i"], c["op_i"]))
    drive_only = {(d["mode"], d["op"]) for d in desc["drives"]} - first
    c_fwd = 2 * len(pairs) + len(drive_only)
    sens = 3 * len(pairs) + len(desc["modes"])
    return c_fwd, sens


def flops(desc, S):
    d = desc["modes"][0]["trunc"]
    D = d ** len(desc["modes"])
    N = desc["n_steps"]
    c_fwd, sens = contraction_counts(desc)
    per = 8.0 * D * S * d              # one contraction over all columns (complex MAC = 8 FLOP)
    fwd = 4 * N * per * c_fwd
    adj = 4 * N * per * (2 * c_fwd + sens)   # recompute + adjoint apply + sensitivities
    return fwd, adj


def kernel_flops(desc, S):
    """Algorithmic FLOP of all launches of one forward + adjoint, per kernel:
    forward (C contractions per stage), recompute (C per stage), reverse (C
    reverse-generator contractions and 3 per pair + 1 per mode sensitivity
    contractions per stage); 4 stages per step, 8 D d S FLOP per contraction."""
    d = desc["modes"][0]["trunc"]
    D = d ** len(desc["modes"])
    N = desc["n_steps"]
    c_fwd, sens = contraction_counts(desc)
    per = 4 * N * 8.0 * D * S * d
    return {"forward": per * c_fwd, "recompute": per * c_fwd, "reverse": per * (c_fwd + sens)}


# Source files that define each profiled kernel (its own file, the shared
# device building blocks and the structures it reads).
KERNEL_SOURCES = {
    "rk4": ("rk4.hip", "kernel_common.h", "internal.h"),
    "recompute": ("rk4.hip", "kernel_common.h", "internal.h"),
    "adjoint": ("adjoint.hip", "kernel_common.h", "internal.h"),
    "lindblad": ("open_real.hip", "gather.hip", "gather.h", "kernel_common.h", "internal.h"),
    "gather": ("gather.hip", "gather_real.hip", "gather.h", "kernel_common.h", "internal.h"),
}


def kernel_sources_sha(kind):
    """SHA-256 over the sources of one kernel family (names and contents, in order)."""
    h = hashlib.sha256()
    for name in KERNEL_SOURCES[kind]:
        h.update(name.encode())
        h.update(open(os.path.join(ROOT, "paper_2406_18155_amd", "csrc", name), "rb").read())
    return h.hexdigest()


def profile_value(fname, key):
    """A per-launch figure from a counter summary in profiles/ (``key: value``
    lines), or None when the file is missing or the kernel sources changed
    since the counters were taken (its sources_sha256 line)."""
    path = os.path.join(ROOT, "profiles", fname)
    if not os.path.exists(path):
        return None
    kv = {}
    for line in open(path):
        if ":" in line:
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("sources_sha256") != kernel_sources_sha(fname.split("_", 1)[0]):
        return None
    try:
        return float(kv[key])
    except (KeyError, ValueError):
        return None


def measured_traffic(kernel_tag):
    """HBM bytes per launch (FETCH_SIZE + WRITE_SIZE, copy-calibrated)."""
    return profile_value(f"{kernel_tag}_traffic.txt", "hbm_bytes_per_launch")


def executed_flop(kernel_tag):
    """FP32 FLOP per launch the kernel executes (VALU FMA and MFMA counters)."""
    return profile_value(f"{kernel_tag}_counters.txt", "executed_fp32_flop_per_launch")


def plain64_forward_ms(scp, si, torch, desc, S):
    """One forward of the workload on the plain complex FP64 path (ms)."""
    g = scp.System(desc)
    psi0 = scp.basis_columns(g.D, desc["columns"], dtype=torch.complex128)
    o = g.opts(S, precision=1)
    ws = g.workspace(o)
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    g.propagate(psi0, opts=o, workspace=ws)
    e1.record(stream)
    torch.cuda.synchronize()
    g.close()
    return e0.elapsed_time(e1)


def serving_leg(scp, si, torch, np, n_req, poisson=True):
    """Continuous-batching replay of the first n_req requests of the mixed
    request stream: saturated, then Poisson at 0.5x and 0.9x saturation, on
    the server's default engine (the batched register-layout kernels); the
    saturated replay again with the small devices' requests batched on the
    gather engine, for comparison."""
    from paper_2406_18155_amd import serve
    reqs = [si.serving_request(r) for r in range(n_req)]
    budget = int(0.5 * torch.cuda.mem_get_info()[0])
    keys = ("p50_s", "p99_s", "mean_s", "makespan_s", "requests_per_s", "steps_dim2_per_s",
            "failed")
    sat = serve.run_stream(reqs, [0.0] * n_req, budget, max_active=64, progress_s=20.0)
    out = {"requests": n_req, "hbm_budget_bytes": budget, "max_active": 64, "engine": "register",
           "saturated": {k: sat[k] for k in keys}}
    if n_req <= 512:
        gat = serve.run_stream(reqs, [0.0] * n_req, budget, max_active=64, engine="auto",
                               progress_s=20.0)
        out["saturated_gather_routing"] = {k: gat[k] for k in keys}
    if not poisson:
        return out
    for frac in (0.5, 0.9):
        arr = si.poisson_arrivals(n_req, frac * sat["requests_per_s"])
        r = serve.run_stream(reqs, arr, budget, max_active=64, progress_s=20.0)
        out[f"poisson_{frac}x"] = {k: r[k] for k in keys}
    # the same requests alone, FP32 fused path against the plain FP64 path
    # (forward only: the FP64 path has no adjoint), on a bounded sample
    n_cmp = min(6, n_req)
    t32, t64 = [], []
    stream = torch.cuda.current_stream()
    for q in reqs[:n_cmp]:
        g = scp.System(q)
        S = len(q["columns"])
        for prec, dt, acc in ((0, torch.complex64, t32), (1, torch.complex128, t64)):
            psi0 = scp.basis_columns(g.D, q["columns"], dtype=dt)
            o = g.opts(S, precision=prec)
            ws = g.workspace(o)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            g.propagate(psi0, opts=o, workspace=ws)
            e1.record(stream)
            torch.cuda.synchronize()
            acc.append(e0.elapsed_time(e1))
        g.close()
    out["fp32_vs_fp64"] = {"requests": n_cmp, "what": "forward of each of the first requests "
                           "alone; the FP64 path has no adjoint",
                           "fp32_ms": sum(t32), "fp64_ms": sum(t64),
                           "speedup": sum(t64) / sum(t32)}
    grads = sum(1 for q in reqs if q["want_grad"])
    out["mix"] = (f"first {n_req} requests of the mixed stream: 2-6 modes, d in {{3,4,5}}, "
                  f"D <= 3125, S = 2^modes, T in [20,200] ns at 50 steps/ns, "
                  f"{grads} with gradient")
    return out


def probe_lines(scp, torch, np, n_wg=1024, iters=2000):
    """The register-layout stepper's d = 3 contraction in its VALU form and in
    two v_mfma_f32_4x4x1f32 forms (with the operand builds and register moves
    the layout needs; issue only), timed on the device.  Algorithmic work:
    9 fibres x 9 complex multiply-adds x 8 FLOP per lane and application."""
    rng = np.random.default_rng(5)
    a = rng.normal(size=(16, 3, 3)) + 1j * rng.normal(size=(16, 3, 3))
    h = 0.1 * (a + a.conj().transpose(0, 2, 1))
    ops = torch.tensor(np.concatenate([h.real.reshape(16, 9), h.imag.reshape(16, 9)], axis=1),
                       dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream()
    flop = n_wg * 256.0 * iters * 648
    names = {0: "VALU FMA (the stepper's form)",
             1: "MFMA 4x4x1 f32, operands built per application, outputs moved to the layout",
             2: "MFMA 4x4x1 f32, operands built once, accumulators in place (issue and padding only)"}
    lines, ref = [], None
    for form in (0, 1, 2):
        o = ops[:1] if form == 2 else ops
        out = scp.probe_contraction(form, o, iters, n_wg)
        ts = []
        for rep in range(3):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            scp.probe_contraction(form, o, iters, n_wg, out=out)
            e1.record(stream)
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        ms = min(ts)
        lines.append({"config": "contraction probe (d = 3, 27 amplitudes per lane)", "form": form,
                      "what": names[form], "n_wg": n_wg, "iters": iters, "ms": ms,
                      "algorithmic_tflops": flop / (ms * 1e-3) / 1e12,
                      "frac_of_157.3": flop / (ms * 1e-3) / 157.3e12})
    return lines


def other_configs(scp, si, torch, np, only=None, plain64=True):
    """Configs 1-3 and the X^6 chain on the GPU: forward and gradient times,
    rate, FP64 forward, and parity against the stored oracle results where
    they exist (one JSON line per config; not part of the default run)."""
    import copy
    lines = []
    cases = [("config1: 2 transmons d=4, full 16x16 U, T=40 ns, 2000 steps", si.config1(), None),
             ("config2/3: 4-fluxonium chain d=5, 16 columns, T=100 ns, 5000 steps, 58 params",
              si.config3(), os.path.join(ROOT, "tests", "golden", "config3_oracle.json")),
             ("x6: 6-fluxonium multipath chain d=4 (D=4096), 64 columns, X on every qubit, "
              "T=50 ns, 5000 steps of 0.01 ns, 148 params (the paper's X^6 benchmark shape; "
              "the paper: forward 2.02 s, gradient 8.55 s on a 32-core CPU, Trotter Q2 + LCAM)",
              si.fluxonium6_x6(), None)]
    if only is not None:
        cases = [c for c, key in zip(cases, ("config1", "chain", "x6")) if key == only]
    stream = torch.cuda.current_stream()

    def timed_gradient(g, psi0, tgt, S):
        """Forward with checkpoints, then fidelity + adjoint: min of 3 each,
        on the engine the system is set to."""
        opts = g.opts(S, with_ckpt=1)
        ws = g.workspace(opts, with_grad=True)
        cot = torch.empty_like(psi0)
        res = []
        for rep in range(3):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
            ev[0].record(stream)
            U = g.propagate(psi0, opts=opts, workspace=ws)
            ev[1].record(stream)
            F, _ = scp.fidelity(U, tgt, cotangent=cot)
            grad = g.adjoint(cot, opts, ws)
            ev[2].record(stream)
            torch.cuda.synchronize()
            res.append((ev[0].elapsed_time(ev[1]), ev[1].elapsed_time(ev[2])))
        eng = g.engine(opts, with_grad=True)
        del ws
        return min(r[0] for r in res), min(r[1] for r in res), F, grad, U, cot, eng

    for name, desc, ref_path in cases:
        g = scp.System(desc)
        S = len(desc["columns"])
        psi0 = scp.basis_columns(g.D, desc["columns"])
        tgt = scp.Target(desc["comp_rows"], desc["comp_cols"], desc["target"])
        fwd_ms, grad_ms, F, grad, U, cot, eng = timed_gradient(g, psi0, tgt, S)
        other = None
        if eng == "gather":
            # the same on the register-layout stepper, for comparison
            g.set_engine("register")
            r_fwd, r_grad, r_F, r_g, _, _, _ = timed_gradient(g, psi0, tgt, S)
            other = {"forward_ms": r_fwd, "fidelity_and_gradient_ms": r_grad, "F": r_F,
                     "grad": r_g}
            g.set_engine("auto")
        # forward alone (no checkpoints: the gather engine where the system
        # has few columns of a small device)
        fo = []
        for rep in range(3):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record(stream)
            Uf = g.propagate(psi0)
            ev[1].record(stream)
            torch.cuda.synchronize()
            fo.append(ev[0].elapsed_time(ev[1]))
        Ff, _ = scp.fidelity(Uf, tgt)
        N = desc["n_steps"]
        fwd_flop, adj_flop = flops(desc, S)
        # the plain FP64 path (one launch per local term) only for the small devices
        p64 = plain64_forward_ms(scp, si, torch, desc, S) if g.D <= 1000 and plain64 else None
        out = {"config": name, "engine": eng, "forward_ms": fwd_ms,
               "fidelity_and_gradient_ms": grad_ms,
               "forward_only_ms": min(fo), "F_forward_only": Ff,
               "O_t": (fwd_ms + grad_ms) / min(fo),
               "steps_dim2_per_s_forward": N * g.D * S / (fwd_ms * 1e-3),
               "forward_tflops": fwd_flop / (fwd_ms * 1e-3) / 1e12,
               "plain_fp64_forward_ms": p64, "F": F, "n_params": len(grad)}
        # plain and phase-compensated fidelity of the same U (wall time of the
        # calls, each synchronising: gather on the device, phase search on the host)
        nq = int(round(np.log2(len(desc["comp_rows"]))))
        if 2 ** nq == len(desc["comp_rows"]) and nq <= 6:
            tf = []
            for fn in (lambda: scp.fidelity(U, tgt, cotangent=cot),
                       lambda: scp.fidelity_zcomp(U, tgt, nq, cotangent=cot)):
                fn()
                t0 = time.perf_counter()
                for _ in range(10):
                    r = fn()
                tf.append((time.perf_counter() - t0) / 10 * 1e3)
            out.update({"fidelity_ms": tf[0], "fidelity_zcomp_ms": tf[1], "F_zcomp": r[0]})
        if ref_path and os.path.exists(ref_path):
            ref = json.load(open(ref_path))
            gref = np.array(ref["grad"])
            out.update({"dF": abs(F - ref["F"]),
                        "grad_rel_err": float(np.abs(grad - gref).max() / np.abs(gref).max())})
            if other is not None:
                other["dF"] = abs(other["F"] - ref["F"])
                other["grad_rel_err"] = float(np.abs(other["grad"] - gref).max() /
                                              np.abs(gref).max())
        if other is not None:
            other.pop("grad")
            out["register_engine"] = other
        g.close()
        lines.append(out)
    if only is None:
        lines.append(static_spectrum_line(scp, np))
        lines += trotter_lines(scp, si, torch, np)
    return lines


def trotter_flop(desc, order):
    """(algorithmic, executed) FP64 FLOP of one product-formula propagation.
    Algorithmic: every local term applied as in App. A, a d x d (single-mode)
    or d^2 x d^2 (pair) complex matrix on every fibre of a column, 8 FLOP per
    complex multiply-add.  Executed: after the library's fusion, which merges
    adjacent couplings on the same ordered mode pair and, when pair gates run
    split (32 D bytes fit in 160 KiB and D / d^2 < 512 fibres), absorbs every
    coupled mode's single-mode gate into a pair operation.  (Where pair gates
    run in place, single-mode gates are applied in registers next to them:
    fewer passes over the state, the same arithmetic.)  Where every mode couples
    through one operator, the pair gates are diagonal in its eigenbasis: one
    d x d matrix per mode and one phase (6 FLOP) per amplitude and piece."""
    d = desc["modes"][0]["trunc"]
    M = len(desc["modes"])
    pairs = [(c["i"], c["j"]) for c in desc["couplings"]]
    E = len(pairs)
    D = d ** M
    passes = {"q1": 1, "q2": 2, "q4": 6, "q4j": 4}[order]   # passes over the terms per step
    units = desc["n_steps"] * len(desc["columns"]) * passes * 8.0
    alg = units * (M * D * d + E * D * d * d)
    ends = {(c["i"], c["op_i"]) for c in desc["couplings"]} | {(c["j"], c["op_j"])
                                                               for c in desc["couplings"]}
    if E > 0 and len(ends) == len({m for m, _ in ends}):
        pieces = {"q1": 1, "q2": 1, "q4": 3, "q4j": 2}[order]
        return alg, desc["n_steps"] * len(desc["columns"]) * pieces * (8.0 * M * D * d + 6.0 * D)
    runs = sum(1 for e in range(E) if e == 0 or pairs[e] != pairs[e - 1])
    absorb = E > 0 and 32 * D <= 160 * 1024 and D // (d * d) < 512
    coupled = {m for p in pairs for m in p}
    lone = M - (len(coupled) if absorb else 0)
    exe = units * (runs * D * d * d + lone * D * d)
    return alg, exe


def trotter_lines(scp, si, torch, np, orders=("q1", "q2", "q4", "q4j"), only=None):
    """Suzuki-Trotter product formulas on the 8-transmon ring (D = 6561, 256
    columns, 3000 steps), the 4-fluxonium chain (D = 625, 16 columns, 5000
    steps) and the 6-fluxonium X^6 chain (D = 4096, 64 columns, 5000 steps):
    call time (gate exponentials + propagation, HIP events on the
    launch stream), algorithmic FP64 rate against the 78.6 TFLOP/s vector
    peak, distance to the FP32 RK4 result, and the oracle on a bounded
    sample (the ring's first 10 steps, 8 columns)."""
    from oracle import trotter as otr
    from oracle.system import OracleSystem
    out = []
    stream = torch.cuda.current_stream()
    for name, desc, ords in (("ring8_d3: 8-transmon ring d=3, D=6561, 256 columns, 3000 steps",
                              si.config5(), orders),
                             ("chain4_d5: 4-fluxonium chain d=5, D=625, 16 columns, 5000 steps",
                              si.config2(), ("q2", "q4")),
                             ("x6_chain6_d4: 6-fluxonium multipath chain d=4, D=4096, 64 columns, "
                              "T=50 ns, 5000 steps of 0.01 ns (the paper's X^6 benchmark shape)",
                              si.fluxonium6_x6(), ("q2",))):
        if only is not None and not name.startswith(only):
            continue
        g = scp.System(desc)
        S = len(desc["columns"])
        psi0 = scp.basis_columns(g.D, desc["columns"], dtype=torch.complex128)
        rk = g.propagate(scp.basis_columns(g.D, desc["columns"])).to(torch.complex128)
        for order in ords:
            ws = torch.empty(g.trotter_workspace_bytes(order), dtype=torch.uint8, device="cuda")
            U = g.propagate_trotter(psi0, order, workspace=ws)
            ms = []
            for _ in range(3):
                ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                ev[0].record(stream)
                U = g.propagate_trotter(psi0, order, workspace=ws)
                ev[1].record(stream)
                torch.cuda.synchronize()
                ms.append(ev[0].elapsed_time(ev[1]))
            t = min(ms)
            alg, exe = trotter_flop(desc, order)
            out.append({"config": "trotter " + name, "order": order, "call_ms": t,
                        "steps_columns_per_s": desc["n_steps"] * S / (t * 1e-3),
                        "algorithmic_fp64_tflops": alg / (t * 1e-3) / 1e12,
                        "executed_fp64_tflops": exe / (t * 1e-3) / 1e12,
                        "frac_fp64_peak": exe / (t * 1e-3) / 78.6e12,
                        "max_abs_diff_vs_rk4_fp32": float((U - rk).abs().max()),
                        "workspace_mib": ws.numel() / 2 ** 20})
            # the LCAM gradient (Sec. 2.5) for a seeded costate: time overhead
            # and memory overhead against the forward alone (where a column and
            # its costate fit in LDS)
            if order in ("q2", "q4") and 16 * (2 * g.D + 512) <= 160 * 1024:
                rng = np.random.Generator(np.random.PCG64(2406018155 + 93))
                lam = rng.normal(size=(S, g.D)) + 1j * rng.normal(size=(S, g.D))
                cot = torch.tensor(lam, dtype=torch.complex128, device="cuda")
                wsa = torch.empty(g.trotter_adjoint_workspace_bytes(order, S), dtype=torch.uint8,
                                  device="cuda")
                g.trotter_adjoint(psi0, cot, order, workspace=wsa)
                ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                ev[0].record(stream)
                g.trotter_adjoint(psi0, cot, order, workspace=wsa)
                ev[1].record(stream)
                torch.cuda.synchronize()
                ta = ev[0].elapsed_time(ev[1])
                # the same gradient started from the forward's result (the
                # walk without the gradient call's own forward)
                g.trotter_adjoint_final(U, cot, order, workspace=wsa)
                ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                ev[0].record(stream)
                g.trotter_adjoint_final(U, cot, order, workspace=wsa)
                ev[1].record(stream)
                torch.cuda.synchronize()
                tf = ev[0].elapsed_time(ev[1])
                # forward run: psi0, psi_T and its workspace; gradient run: psi0,
                # the cotangent and its workspace, inside which it runs its own
                # forward (the forward's workspace is not needed beside it)
                fwd_bytes = 2 * psi0.numel() * psi0.element_size() + ws.numel()
                grad_bytes = 2 * psi0.numel() * psi0.element_size() + wsa.numel()
                out[-1].update({"lcam_gradient_ms": ta, "lcam_O_t": (t + ta) / t,
                                "lcam_from_final_ms": tf, "lcam_O_t_from_final": (t + tf) / t,
                                "lcam_O_m": grad_bytes / fwd_bytes,
                                "lcam_note": "gradient call (forward, then the reverse-time walk) "
                                             "for a seeded costate; from_final: the call that "
                                             "starts from the forward's psi(T); O_m: "
                                             "gradient-run device bytes / forward-run device "
                                             "bytes"})
                del wsa
            if name.startswith("x6_"):
                out[-1]["paper_forward_s_context"] = 2.02
                out[-1]["paper_context"] = ("SuperGrad Q2 forward of its X^6 task on a 32-core "
                                            "EPYC 7513, truncation not stated (Sec. 4.2 table)")
        g.close()
    if only is not None:
        return out
    # oracle on a bounded sample of the ring
    desc = si.config5()
    cols = np.asarray(desc["columns"])[si.sampled_columns(len(desc["columns"]))]
    o = OracleSystem(desc)
    t0 = time.perf_counter()
    otr.propagate(o, "q2", psi0=np.eye(o.D)[:, cols], n_steps=10)
    dt = time.perf_counter() - t0
    out.append({"config": "trotter oracle (CPU, FP64, q2)", "sample": "ring8_d3, 10 steps x 8 columns",
                "steps_columns_per_s": 10 * len(cols) / dt, "cores": 1})
    return out


def static_spectrum_line(scp, np):
    """Static ZZ of the paper's three-fluxonium multipath chain (Sec. 3.2) at
    d = 4 (D = 64): call times on the GPU path and of the oracle, and the J_C
    that zeroes zeta_ZZI at J_L = 2 MHz from GPU evaluations."""
    from scipy.optimize import brentq
    from oracle.system import OracleSystem
    from oracle.spectrum import static_zz, static_zz_grad
    fix = json.load(open(os.path.join(ROOT, "tests", "golden", "static_zz_paper.json")))

    def chain(jc):
        modes = [{"kind": "fluxonium", "EC": q["EC"] * 2 * math.pi, "EJ": q["EJ"] * 2 * math.pi,
                  "EL": q["EL"] * 2 * math.pi, "phiext": math.pi, "basis_dim": 80, "trunc": 4}
                 for q in fix["fluxonium"]]
        coup = []
        for (i, j) in ((0, 1), (1, 2)):
            coup.append({"i": i, "j": j, "op_i": "n", "op_j": "n", "g": jc * 1e-3 * 2 * math.pi})
            coup.append({"i": i, "j": j, "op_i": "phi", "op_j": "phi",
                         "g": -fix["J_L_MHz"] * 1e-3 * 2 * math.pi})
        return {"modes": modes, "couplings": coup, "drives": [], "T": 1.0, "n_steps": 1}

    g = scp.System(chain(12.0))
    g.static_zz(0, 1, with_grad=True)
    t0 = time.perf_counter()
    for _ in range(10):
        g.static_zz(0, 1, with_grad=True)
    gpu_ms = (time.perf_counter() - t0) / 10 * 1e3
    g.close()
    o = OracleSystem(chain(12.0))
    t0 = time.perf_counter()
    static_zz(o, 0, 1)
    static_zz_grad(o, 0, 1)
    oracle_ms = (time.perf_counter() - t0) * 1e3

    def zg(jc):
        s = scp.System(chain(jc))
        z = s.static_zz(0, 1)
        s.close()
        return z

    return {"config": "static ZZ: paper's 3-fluxonium multipath chain, d=4 (D=64), J_L=2 MHz",
            "static_zz_with_grad_ms": gpu_ms, "oracle_static_zz_with_grad_ms": oracle_ms,
            "J_C_zero_MHz_d4": brentq(zg, 5.0, 20.0, xtol=1e-6),
            "paper_J_C_MHz": fix["J_C_opt_MHz"],
            "note": "the oracle at d=5 gives 12.250 MHz (pinned); d=4 truncates the chain"}


def lindblad_macs(desc):
    """Complex multiply-adds per density-matrix element and RK4 stage of the
    open-system kernel: the static diagonal (1), one relaxation jump per mode
    where both digits can be raised ((d-1)^2/d^2 of the elements), per driven
    mode a d-term contraction on the ket and on the bra digits, per coupled
    mode pair a d^2-term contraction on each side."""
    d = desc["modes"][0]["trunc"]
    M = len(desc["modes"])
    driven = {dr["mode"] for dr in desc["drives"]}
    pairs = {tuple(sorted((c["i"], c["j"]))) for c in desc["couplings"]}
    relax = sum(1 for m in desc["modes"] if m.get("gamma1", 0.0) > 0)
    return 1 + relax * (d - 1) ** 2 / d ** 2 + len(driven) * 2 * d + len(pairs) * 2 * d * d


def lindblad_line(scp, si, torch, np, reps=3):
    """Open-system propagation of the 4-fluxonium chain truncated to d = 3
    (D = 81, the vectorised density matrix has D^2 = 6561 entries), its 256
    computational matrix units, T = 100 ns, 5000 RK4 steps, T1/T_phi per mode:
    call time from HIP events on the launch stream, the channel's average gate
    fidelity, the algorithmic FP32 rate against the vector peak (8 FLOP per
    complex multiply-add of ``lindblad_macs``), and the oracle on a bounded
    sample (one matrix unit, 5 steps)."""
    from oracle import lindblad as olb
    from oracle.system import OracleSystem
    desc = si.open_chain()
    g = scp.System(desc)
    st = [desc["columns"][c] for c in desc["comp_cols"]]
    S = len(st) ** 2
    DD = g.D * g.D
    N = desc["n_steps"]
    rho0 = scp.matrix_units(g.D, st)
    ws = torch.empty(g.lindblad_workspace_bytes(), dtype=torch.uint8, device="cuda")
    rhoT = g.propagate_lindblad(rho0, workspace=ws)
    stream = torch.cuda.current_stream()
    ms = []
    for _ in range(reps):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record(stream)
        g.propagate_lindblad(rho0, rhoT=rhoT, workspace=ws)
        ev[1].record(stream)
        torch.cuda.synchronize()
        ms.append(ev[0].elapsed_time(ev[1]))
    t = min(ms)
    cot = torch.empty_like(rhoT)
    F, _ = scp.fidelity_channel(rhoT, scp.ChannelTarget(desc["comp_rows"], desc["target"]),
                                cotangent=cot)
    # gradient: the adjoint call recomputes the forward with checkpoints, then
    # walks the segments in reverse (drive parameters, couplings, decay rates)
    wsa = torch.empty(g.lindblad_adjoint_workspace_bytes(S), dtype=torch.uint8, device="cuda")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    ev[0].record(stream)
    grad = g.lindblad_adjoint(rho0, cot, workspace=wsa)
    ev[1].record(stream)
    torch.cuda.synchronize()
    tg = ev[0].elapsed_time(ev[1])
    m_fwd = 2 * rho0.numel() * rho0.element_size()
    m_grad = m_fwd + wsa.numel()
    del wsa
    g.close()
    flop = 8.0 * lindblad_macs(desc) * DD * S * 4 * N
    ex = executed_flop("lindblad_open_chain_d3")
    o = OracleSystem(desc)
    t0 = time.perf_counter()
    olb.propagate(o, olb.matrix_units(o.D, st)[:1], n_steps=5)
    dt = time.perf_counter() - t0
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count()
    return {"config": "open system: 4-fluxonium chain d=3 (D=81, D^2=6561), 256 matrix units of "
                      "the 16 computational states, T=100 ns, 5000 RK4 steps, T1/T_phi ~ U[20,60] us",
            "call_ms": t, "F_avg": F,
            "gradient_call_ms": tg, "n_grad_params": int(len(grad)),
            "O_t": tg / t, "O_m": m_grad / m_fwd,
            "O_note": "gradient call (forward with checkpoints + reverse) / forward; "
                      "gradient-run device bytes / forward-only matrix bytes",
            "steps_dim2_per_s": N * DD * S / (t * 1e-3),
            "roofline": {"bound": "alu", "achieved": flop / (t * 1e-3) / 1e12, "peak": 157.3,
                         "unit": "TFLOP/s", "frac": flop / (t * 1e-3) / PEAK_FP32,
                         "traffic": measured_traffic("lindblad_open_chain_d3"),
                         "kernel": "l_rk4_kernel<3,4,true,false>", "algorithmic_flop": flop,
                         "executed_tflops": None if ex is None else ex / (t * 1e-3) / 1e12,
                         "executed_frac": None if ex is None else ex / (t * 1e-3) / PEAK_FP32},
            "cpu_oracle": {"steps_dim2_per_s": 5 * DD / dt, "cores": cores,
                           "sample": "1 matrix unit, 5 of 5000 steps, dense numpy FP64"}}


def sampled_desc(si, np):
    desc = si.config5()
    samp = si.sampled_columns(len(desc["columns"]), 8)
    full_t = desc["target"]
    desc["comp_rows"] = [desc["comp_rows"][j] for j in samp]
    desc["columns"] = [desc["columns"][j] for j in samp]
    desc["comp_cols"] = list(range(len(samp)))
    desc["target"] = full_t[np.ix_(samp, samp)]
    return desc


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _oracle_fwd_grad(si, np, desc, n_steps):
    """Oracle forward + fidelity + adjoint gradient of desc over its first
    n_steps steps (same shapes and per-step work as the full run); seconds."""
    from oracle.system import OracleSystem
    from oracle.rk4 import basis_columns, propagate
    from oracle.fidelity import cotangent, fidelity
    from oracle.adjoint import gradient
    t0 = time.perf_counter()
    s = OracleSystem(desc)
    psi0 = basis_columns(s.D, desc["columns"])
    U = propagate(s, psi0)
    F, tau = fidelity(U, desc["comp_rows"], desc["comp_cols"], desc["target"])
    lam = cotangent(U.shape, desc["comp_rows"], desc["comp_cols"], desc["target"], tau)
    gradient(s, lam, psi0)
    return time.perf_counter() - t0


def _prefix(desc, n_steps):
    """desc cut to its first n_steps steps at the same step h (pulse envelopes
    rescaled; the per-step work does not depend on their values)."""
    import copy
    d = copy.deepcopy(desc)
    scale = n_steps / d["n_steps"]
    d["T"] *= scale
    d["n_steps"] = n_steps
    for dr in d["drives"]:
        dr["sigma"] *= scale
    return d


def cpu_baseline(si, np, steps=10, reps=3):
    """The oracle as written, timed on this host: the 8 seeded sampled columns
    of the benchmark workload over a prefix of ``steps`` RK4 steps, forward +
    fidelity + adjoint gradient; min and median of ``reps`` runs with every
    BLAS thread, and one run with one thread.  The rate per column and step is
    the full workload's (same shapes); the full 256-column, 3000-step time is
    extrapolated by (256/8) x (3000/steps) and labelled so."""
    desc = _prefix(sampled_desc(si, np), steps)
    ts = [_oracle_fwd_grad(si, np, desc, steps) for _ in range(reps)]
    try:
        from threadpoolctl import threadpool_info, threadpool_limits
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
        with threadpool_limits(limits=1):
            t1 = _oracle_fwd_grad(si, np, desc, steps)
    except Exception:
        cores, t1 = os.cpu_count(), None
    D, S = 3 ** 8, len(desc["columns"])
    tmin, tmed = min(ts), float(np.median(ts))
    full = si.config5()
    return {"value": steps * D * S / tmin, "unit": "steps*dim^2/s", "cores": cores,
            "kind": "oracle",
            "sample": f"8-transmon ring, the 8 seeded sampled columns, first {steps} of 3000 RK4 "
                      f"steps, forward + fidelity + adjoint gradient (40 params), numpy FP64; "
                      f"min of {reps} = {tmin:.2f} s, median {tmed:.2f} s",
            "median_value": steps * D * S / tmed,
            "one_thread_value": None if t1 is None else steps * D * S / t1,
            "cpu_model": cpu_model(), "os_cpu_count": os.cpu_count(),
            "extrapolated_full_workload_s": tmin * (len(full["columns"]) / S) *
                                            (full["n_steps"] / steps),
            "extrapolation": "x 256/8 columns x 3000/steps steps (labelled estimate)"}


def cpu_protocol(si, np):
    """The oracle's timing protocol in full (long: tens of minutes): configs 1
    and 2/3 over all their steps (forward + fidelity + gradient), min of 3 and
    median with every BLAS thread, one run with one thread; config 5 on its 8
    sampled columns over 300 steps, extrapolated to the full run."""
    from threadpoolctl import threadpool_limits
    out = []
    cases = [("config1: 2 transmons d=4, 16 columns, 2000 steps", si.config1(), None, 3),
             ("config2/3: 4-fluxonium chain d=5, 16 columns, 5000 steps", si.config3(), None, 3),
             ("config5 sampled: 8-transmon ring d=3, 8 sampled columns, 300 of 3000 steps",
              sampled_desc(si, np), 300, 3)]
    for name, desc, n, reps in cases:
        d = desc if n is None else _prefix(desc, n)
        ts = [_oracle_fwd_grad(si, np, d, d["n_steps"]) for _ in range(reps)]
        with threadpool_limits(limits=1):
            t1 = _oracle_fwd_grad(si, np, d, d["n_steps"])
        D = desc["modes"][0]["trunc"] ** len(desc["modes"])
        S = len(desc["columns"])
        line = {"config": name, "min_s": min(ts), "median_s": float(np.median(ts)),
                "one_thread_s": t1, "steps_dim2_per_s": d["n_steps"] * D * S / min(ts),
                "cpu_model": cpu_model(), "os_cpu_count": os.cpu_count()}
        if n is not None:
            line["extrapolated_full_256_columns_s"] = min(ts) * 32 * desc["n_steps"] / n
        out.append(line)
        print(json.dumps(line), flush=True)
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-check", action="store_true")
    ap.add_argument("--no-plain64", action="store_true")
    ap.add_argument("--serve-requests", type=int, default=128)
    ap.add_argument("--serve-only", type=int, default=0,
                    help="only replay the first N requests of the serving stream saturated (also "
                         "with gather routing when N <= 512) and exit")
    ap.add_argument("--configs", action="store_true",
                    help="only time configs 1-3 (one JSON line each) and exit")
    ap.add_argument("--config-only", choices=("config1", "chain", "x6"), default=None,
                    help="with --configs: only this case (config1; chain: the 4-fluxonium "
                         "chain of configs 2/3; x6)")
    ap.add_argument("--probe", action="store_true",
                    help="only time the contraction probe (VALU and MFMA forms of the d = 3 "
                         "contraction) and exit")
    ap.add_argument("--trotter", action="store_true",
                    help="only time the Suzuki-Trotter product formulas (one JSON line each) and exit")
    ap.add_argument("--trotter-orders", default="q1,q2,q4,q4j")
    ap.add_argument("--frame", choices=("real", "complex"), default="complex",
                    help="generator evaluation of the timed steps: the rotated complex operators "
                         "(default; its gradient meets the 1e-4 bar at F ~ 1) or the real frame "
                         "(faster; its FP32 gradient near F = 1 is ~2e-4), which the line then "
                         "reports beside the timed one")
    ap.add_argument("--lindblad", action="store_true",
                    help="only time the open-system (Lindblad) propagation (one JSON line) and exit")
    ap.add_argument("--no-lindblad", action="store_true")
    ap.add_argument("--no-product-formula", action="store_true")
    ap.add_argument("--cpu-protocol", action="store_true",
                    help="only run the oracle's full CPU timing protocol (long) and exit")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain 1 GiB device-to-device copy (to scale HBM counters)")
    args = ap.parse_args()
    if args.copy_calibration:
        import torch
        a = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
        b = torch.empty_like(a)
        a.fill_(1)
        b.copy_(a)
        torch.cuda.synchronize()
        b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes": 1 << 30}))
        return
    if args.gpus != 1:
        print("bench.py: runs on one GPU only (the columns would shard across GPUs with no "
              "communication until the final fidelity and gradient sums). Use --gpus 1.",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import scp_inputs as si
    if args.cpu_protocol:
        cpu_protocol(si, np)
        return
    import torch
    import paper_2406_18155_amd as scp

    if args.trotter:
        for line in trotter_lines(scp, si, torch, np, tuple(args.trotter_orders.split(","))):
            print(json.dumps(line), flush=True)
        return
    if args.lindblad:
        print(json.dumps(lindblad_line(scp, si, torch, np)), flush=True)
        return
    if args.serve_only > 0:
        line = serving_leg(scp, si, torch, np, args.serve_only, poisson=False)
        print(json.dumps(line), flush=True)
        return
    if args.probe:
        for line in probe_lines(scp, torch, np):
            print(json.dumps(line), flush=True)
        return
    if args.configs:
        for line in other_configs(scp, si, torch, np, args.config_only, not args.no_plain64):
            print(json.dumps(line), flush=True)
        return
    dev = torch.device("cuda:0")
    desc = si.config5()
    S = len(desc["columns"])
    D = 3 ** 8
    N = desc["n_steps"]
    stream = torch.cuda.current_stream()

    state = {}
    kt = {"forward": [0.0, 0], "recompute": [0.0, 0], "reverse": [0.0, 0]}

    def step(timed_kernels=False):
        g = scp.System(desc)
        g.set_real_frame(args.frame == "real")
        if timed_kernels:
            g.set_timing(True)
        psi0 = scp.basis_columns(g.D, desc["columns"], device=dev)
        opts = g.opts(S, with_ckpt=1)
        if "ws" not in state:
            state["ws"] = g.workspace(opts, with_grad=True)
            state["cot"] = torch.empty_like(psi0)
            state["tgt"] = scp.Target(desc["comp_rows"], desc["comp_cols"], desc["target"])
        ws = state["ws"]
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        ev[0].record(stream)
        U = g.propagate(psi0, opts=opts, workspace=ws)
        ev[1].record(stream)
        F, _ = scp.fidelity(U, state["tgt"], cotangent=state["cot"], sync=False)
        ev[2].record(stream)
        grad = g.adjoint(state["cot"], opts, ws)
        ev[3].record(stream)
        if timed_kernels:
            torch.cuda.synchronize()
            state.setdefault("fwd_ms", []).append(ev[0].elapsed_time(ev[1]))
            state.setdefault("adj_ms", []).append(ev[2].elapsed_time(ev[3]))
            for k, (ms, n) in g.kernel_times().items():
                kt[k][0] += ms
                kt[k][1] += n
        g.close()
        return grad

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step(timed_kernels=True)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / args.steps

    fwd_flop, adj_flop = flops(desc, S)
    kflop = kernel_flops(desc, S)
    fwd_ms = float(np.mean(state["fwd_ms"]))
    adj_ms = float(np.mean(state["adj_ms"]))
    value = N * D * S / dt

    def kernel_line(kind, name, tag, bound_note):
        ms, n = kt[kind]
        launch_ms = ms / n
        flop_launch = kflop[kind] / (n / args.steps)
        ex = executed_flop(tag)
        line = {"bound": "alu", "achieved": flop_launch / (launch_ms * 1e-3) / 1e12,
                "peak": PEAK_FP32 / 1e12, "unit": "TFLOP/s",
                "frac": flop_launch / (launch_ms * 1e-3) / PEAK_FP32,
                "traffic": measured_traffic(tag), "kernel": name,
                "launches_per_step": n / args.steps, "launch_ms": launch_ms,
                "algorithmic_flop_per_launch": flop_launch,
                "executed_tflops": None if ex is None else ex / (launch_ms * 1e-3) / 1e12,
                "executed_frac": None if ex is None else ex / (launch_ms * 1e-3) / PEAK_FP32,
                "share_of_step": ms / args.steps / (dt * 1e3), "note": bound_note}
        return line

    ev = 3 if args.frame == "real" else 2   # evaluation: real frame (1) and parity (2)
    sfx = "" if args.frame == "real" else "_complex"
    kernels = {
        "reverse": kernel_line("reverse", f"adjoint_kernel<3,3,1,{ev}>", "adjoint_ring8_d3" + sfx,
                               "reverse walk of one checkpoint segment: per stage C reverse "
                               "contractions + (3 per pair + 1 per mode) sensitivity contractions"),
        "forward": kernel_line("forward", f"rk4_kernel<3,3,1,false,{ev}>", "rk4_ring8_d3" + sfx,
                               "the whole 3000-step forward in one launch, C contractions per stage"),
        "recompute": kernel_line("recompute", f"rk4_kernel<3,3,1,true,{ev}>",
                                 "recompute_ring8_d3" + sfx,
                                 "one checkpoint segment forward, stage inputs stored"),
    }

    # parity on the same run, in the benchmark's launch configuration
    parity = {}
    if not args.no_check:
        st_path = os.path.join(ROOT, "tests", "golden", "config5_state_oracle.json")
        cz_path = os.path.join(ROOT, "tests", "golden", "config5_sampled_oracle.json")
        g = scp.System(desc)
        g.set_real_frame(args.frame == "real")
        psi0 = scp.basis_columns(g.D, desc["columns"], device=dev)
        opts = g.opts(S, with_ckpt=1)
        ws = state["ws"]
        U = g.propagate(psi0, opts=opts, workspace=ws)
        cot = state["cot"]
        samp = si.sampled_columns(S, 8)
        gc_ = None
        if os.path.exists(st_path):
            ref = json.load(open(st_path))
            phi = np.load(os.path.join(ROOT, "tests", "golden", "config5_state_target.npy"),
                          allow_pickle=False)
            F, _ = scp.fidelity_states(U, scp.StateTarget(samp, phi.T), cotangent=cot)
            gr = g.adjoint(cot, opts, ws)
            gref = np.array(ref["grad"])
            parity.update({"F": F, "dF": abs(F - ref["F"]),
                           "grad_rel_err": float(np.abs(gr - gref).max() / np.abs(gref).max()),
                           "parity_sample": "all 256 columns propagated; composite state cost "
                                            "of the 8 seeded sampled columns against stored "
                                            "targets near the oracle's own final states "
                                            "(F_oracle = %.6f) vs the stored FP64 oracle" % ref["F"]})
            # the other evaluation of the generator on the same target (the real
            # frame's FP32 gradient near F = 1 is above the 1e-4 bar)
            gc_ = scp.System(desc)
        if gc_ is not None:
            other = args.frame != "real"
            gc_.set_real_frame(other)
            Uc = gc_.propagate(psi0, opts=opts, workspace=ws)
            Fc, _ = scp.fidelity_states(Uc, scp.StateTarget(samp, phi.T), cotangent=cot)
            grc = gc_.adjoint(cot, opts, ws)
            tag = "real_frame" if other else "complex_eval"
            parity.update({f"dF_{tag}": abs(Fc - ref["F"]),
                           f"grad_rel_err_{tag}":
                               float(np.abs(grc - gref).max() / np.abs(gref).max())})
            # one timed step of the other evaluation, for context
            ms_other = []
            for rep in range(2):
                go = scp.System(desc)
                go.set_real_frame(other)
                torch.cuda.synchronize()
                t0o = time.perf_counter()
                Uo = go.propagate(psi0, opts=opts, workspace=ws)
                scp.fidelity(Uo, state["tgt"], cotangent=cot, sync=False)
                go.adjoint(cot, opts, ws)
                torch.cuda.synchronize()
                ms_other.append((time.perf_counter() - t0o) * 1e3)
                go.close()
            parity[f"ms_per_step_{tag}"] = min(ms_other)
            parity[f"value_{tag}"] = N * D * S / (min(ms_other) * 1e-3)
            gc_.close()
            U = g.propagate(psi0, opts=opts, workspace=ws)
        if os.path.exists(cz_path):
            ref = json.load(open(cz_path))
            sd = sampled_desc(si, np)
            F2, _ = scp.fidelity(U, scp.Target(sd["comp_rows"], samp, sd["target"]),
                                 cotangent=cot)
            g2 = g.adjoint(cot, opts, ws)
            gref = np.array(ref["grad"])
            parity.update({"F_cz_sampled": F2, "dF_cz_sampled": abs(F2 - ref["F"]),
                           "grad_rel_err_cz_sampled":
                               float(np.abs(g2 - gref).max() / np.abs(gref).max())})
        g.close()

    m_fwd = 2 * S * D * 8
    g = scp.System(desc)
    m_grad = m_fwd + g.workspace_bytes(g.opts(S, with_ckpt=1), with_grad=True)
    g.close()

    out = {
        "metric": "RK4 steps*dim^2/s (forward + adjoint gradient)",
        "value": value,
        "unit": "steps*dim^2/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": dt * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64",
        "data": "synthetic",
        "config": {"workload": "8-transmon ring, d=3, D=6561, 256 computational columns, "
                               "T=60 ns, 3000 RK4 steps, 40 gradient parameters",
                   "global_batch": S, "seq_len": N,
                   "generator_evaluation": ("real frame (real operators between diagonal "
                                            "frame rotations)" if args.frame == "real" else
                                            "complex (rotated operators per half step)")},
        # the dominant kernel (HIP events recorded by the library on the launch stream)
        "roofline": kernels["reverse"],
        "kernels": kernels,
        "forward": {"ms": fwd_ms, "steps_dim2_per_s": N * D * S / (fwd_ms * 1e-3),
                    "tflops": fwd_flop / (fwd_ms * 1e-3) / 1e12,
                    "frac": fwd_flop / (fwd_ms * 1e-3) / PEAK_FP32},
        # per segment a recompute launch and a reverse launch; algorithmic work of the call
        "adjoint": {"ms": adj_ms, "tflops": adj_flop / (adj_ms * 1e-3) / 1e12,
                    "frac": adj_flop / (adj_ms * 1e-3) / PEAK_FP32,
                    "algorithmic_flop": adj_flop},
        "O_t": (fwd_ms + adj_ms) / fwd_ms,
        "O_m": m_grad / m_fwd,
        "O_m_note": "gradient-run device bytes (states + workspace) / forward-only state bytes",
    }
    out.update(parity)
    if not args.no_plain64:
        p64 = plain64_forward_ms(scp, si, torch, desc, S)
        out["plain_fp64"] = {"forward_ms": p64, "speedup_fused_fp32_forward": p64 / fwd_ms,
                             "path": "complex FP64, one launch per local term"}
    if args.serve_requests > 0:
        out["serving"] = serving_leg(scp, si, torch, np, args.serve_requests)
    if not args.no_lindblad:
        out["open_system"] = lindblad_line(scp, si, torch, np)
    if not args.no_product_formula:
        out["product_formula"] = trotter_lines(scp, si, torch, np, ("q2",), only="chain4_d5")[0]
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(si, np)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
