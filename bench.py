#!/usr/bin/env python3
"""Benchmark: Hamiltonian nonzeros per second on one MI355X.

One step is the whole construction path for one problem, starting from the
problem description and the two-body table resident in HBM:
    ci_basis_build       (size query, arena, tables, partner lists)
    ci_hamiltonian_count (count + scan; one sync to read nnz)
    ci_hamiltonian_fill  (col/val of every stored entry)
    ci_hamiltonian_vjp   (adjoint onto the table, upstream G_e = psi_i psi_j;
                          recomputes the pair and phase structure)
(--adjoint stored: ci_hamiltonian_fill_keys + ci_hamiltonian_vjp_keys, where
the fill stores one structure word per entry and the adjoint reads them.)
value = nnz / (seconds per step).  The default workload is 10B, Z = N = 5,
Nmax = 4, 2M = 0, positive parity (D = 581,740, 143.9 M stored entries):
forward + adjoint.

The JSON line also carries per-stage times, forward and adjoint legs each
with nonzeros/s, an HBM roofline from the algorithmic bytes (timed with HIP
events on the stream the kernels run on) and a VALU issue fraction from the
committed counters, the 6Li Nmax = 6 workload, the batched mode (64 bases,
fill + adjoint captured in one HIP graph), the eigensolver on the full and on
the stored upper-triangle matrix, and the FP64 oracle timed on the host cores
on a bounded sample of rows.
"""
from __future__ import annotations

import argparse
import glob
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def ensure_library():
    import paper_1412_5989_amd as ci

    if not os.path.exists(ci.LIB_PATH):
        from paper_1412_5989_amd import build

        build.build_library()
    ci.load_library()
    return ci


class EventTimer:
    """Accumulates HIP-event durations of one kernel family on one stream."""

    def __init__(self, torch, stream):
        self.torch, self.stream, self.pairs = torch, stream, []

    def __enter__(self):
        self.a = self.torch.cuda.Event(enable_timing=True)
        self.b = self.torch.cuda.Event(enable_timing=True)
        self.a.record(self.stream)
        return self

    def __exit__(self, *exc):
        self.b.record(self.stream)
        self.pairs.append((self.a, self.b))

    def mean_ms(self):
        self.torch.cuda.synchronize()
        return float(np.mean([a.elapsed_time(b) for a, b in self.pairs])) if self.pairs else 0.0


# launch shapes that a kernel's counters depend on
FILL_SHAPE = ("row_waves", "row_grab", "row_xcd")
ADJ_SHAPE = ("adj_rows", "adj_tile_n", "adj_persistent", "row_xcd", "adj_wide", "adj_flush")
ADJK_SHAPE = ("adjk_rows", "adjk_tile_n", "adjk_persistent", "row_xcd", "adj_flush")


def measured_counters(profile: str, shape=None):
    """Per-launch figures from a committed counter summary under profiles/
    (lines "name: value"), or None when the kernel source named in it has
    changed since the counters were taken (its SHA-256 no longer matches), or
    when they were taken at other launch shapes than `shape` (a dict; the
    summary names its own as launch_shape: name=value,...)."""
    path = os.path.join(ROOT, "profiles", profile)
    if not os.path.exists(path):
        return None
    fields = {}
    with open(path) as f:
        for line in f:
            if ":" in line and not line.startswith(("|", "#", " ")):
                k, v = line.split(":", 1)
                fields[k.strip()] = v.strip()
    files = fields.get("kernel_source_files", "kernels.hip ci_internal.h").split()
    csrc = os.path.join(ROOT, "paper_1412_5989_amd", "csrc")
    try:
        digest = hashlib.sha256(b"".join(open(os.path.join(csrc, f), "rb").read() for f in files)).hexdigest()
    except OSError:
        return None
    if fields.get("kernel_source_sha256") != digest:
        return None
    if shape is not None:
        taken = dict(kv.split("=") for kv in fields.get("launch_shape", "").split(",") if kv)
        if any(taken.get(k) != str(v) for k, v in shape.items()):
            return None
    out = {}
    for k in ("traffic_bytes_per_launch", "valu_insts_per_launch"):
        if k in fields:
            out[k] = int(float(fields[k]))
    return out


def cpu_baseline(problem, tbme_seed, psi_seed, budget_s=15.0):
    """The FP64 oracle on sampled rows: forward rows + their gradient."""
    import oracle
    import seeded_inputs as si

    o = oracle.Oracle(oracle.Problem(*problem))
    o.set_tbme(si.tbme_f32(tbme_seed, o.n_tbme).astype(np.float64))
    ps = si.psi(psi_seed, o.dim)

    def run(nrows, seed):
        rows = si.sample_rows(o.dim, nrows, seed)
        t0 = time.perf_counter()
        counts, cols, _ = o.rows(rows)
        G = si.upstream_grad(ps, np.repeat(rows, counts), cols).astype(np.float64)
        o.grad_rows(rows, G)
        return int(counts.sum()), time.perf_counter() - t0, len(rows)

    run(64, 1)  # warm-up (threads, caches)
    n, t, nr = run(256, 3)
    nrows = int(min(o.dim, max(256, nr * budget_s / max(t, 1e-3))))
    n, t, nr = run(nrows, 2)
    threads = oracle.max_threads()
    # the same on one thread, on a smaller sample (~3 s)
    oracle.set_threads(1)
    try:
        _, tp, np_ = run(64, 5)  # probe, then ~3 s
        n1, t1, nr1 = run(int(min(o.dim, max(64, np_ * 3.0 / max(tp, 1e-3)))), 4)
    finally:
        oracle.set_threads(threads)
    return {
        "value": n / t,
        "unit": "nonzeros/s",
        "cores": threads,
        "kind": "oracle",
        "sample": "%d sampled rows of the same workload (%d stored entries), row scan + values on %d "
                  "OpenMP threads, gradient of those rows on 1 thread, %.1f s" % (nr, n, threads, t),
        "value_1_thread": n1 / t1,
        "sample_1_thread": "%d sampled rows (%d stored entries), %.1f s" % (nr1, n1, t1),
    }


def copy_calibration(torch, mib):
    """A plain device-to-device copy of known size, three times (to scale
    hardware byte counters under rocprofv3)."""
    if mib > 0:
        src = torch.ones(mib * (1 << 20) // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst


def run_lanczos(ci, torch, prob, tbme_seed):
    """The step after construction: full symmetric CSR, H x, lowest eigenpair."""
    import seeded_inputs as si

    b = ci.ci_basis_build([prob])
    D = b.info[0]["dim"]
    tb = torch.from_numpy(si.tbme_f32(tbme_seed, b.n_tbme)).cuda()
    rp, nnz = ci.ci_hamiltonian_count_full(b)
    col, val = ci.ci_hamiltonian_fill_full(b, tb, rp)
    stream = torch.cuda.current_stream()
    ev = EventTimer(torch, stream)
    for _ in range(3):
        with ev:
            ci.ci_hamiltonian_fill_full(b, tb, rp, col, val)
    fill_ms = ev.mean_ms()
    x = torch.ones(D, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    ci.ci_hamiltonian_spmv(b, 0, rp, col, val, x, y)
    es = EventTimer(torch, stream)
    for _ in range(10):
        with es:
            ci.ci_hamiltonian_spmv(b, 0, rp, col, val, x, y)
    spmv_ms = es.mean_ms()
    # algorithmic bytes of H x: col + val per entry, row_ptr per row, x read
    # once and y written once
    alg = 8 * nnz[0] + 8 * (D + 1) + 16 * D
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    E, v, it = ci.ci_lanczos(b, 0, rp, col, val, max_iter=300, tol=1e-12)
    t_l = time.perf_counter() - t0
    del col, val
    # the same on the construction's own output, the stored upper triangle:
    # every stored entry read once for both y_i and y_j (the transposed half
    # by FP64 device atomics)
    rpu, nnzu = ci.ci_hamiltonian_count(b)
    colu, valu = ci.ci_hamiltonian_fill(b, tb, rpu)
    eu = EventTimer(torch, stream)
    for _ in range(10):
        with eu:
            ci.ci_hamiltonian_spmv_upper(b, 0, rpu, colu, valu, x, y)
    spmv_u_ms = eu.mean_ms()
    alg_u = 8 * nnzu[0] + 8 * (D + 1) + 16 * D
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    Eu, _, itu = ci.ci_lanczos_upper(b, 0, rpu, colu, valu, max_iter=300, tol=1e-12)
    t_lu = time.perf_counter() - t0
    b.free()
    return {"nnz_full": nnz[0], "fill_full_ms": fill_ms, "fill_full_nnz_per_s": nnz[0] / (fill_ms * 1e-3),
            "spmv_ms": spmv_ms, "spmv_GBps": alg / (spmv_ms * 1e-3) / 1e9,
            "spmv_frac_of_hbm_peak": alg / (spmv_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
            "lanczos_s": t_l, "lanczos_iters": it, "lowest_eigenvalue_MeV": E,
            "upper": {"operand": "stored upper triangle (ci_hamiltonian_fill output)", "nnz": nnzu[0],
                      "spmv_ms": spmv_u_ms,
                      "spmv_roofline": {"bound": "hbm", "achieved": alg_u / (spmv_u_ms * 1e-3) / 1e9,
                                        "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                        "frac": alg_u / (spmv_u_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                                        "alg_bytes_per_launch": alg_u},
                      "lanczos_s": t_lu, "lanczos_iters": itu, "lowest_eigenvalue_MeV": Eu}}


def threebody_block_elements(t, req):
    """Coupled elements each request depends on: the (J, T) blocks of its
    triple pair with |M| <= J and |M_T| <= T, nb x nk elements each
    (the row of D^T, block of A, column of D of paper Sec. 3.1)."""
    q = req % t.n_sps
    j = t.nlj[t.morb[q, 0], 2].astype(np.int64)
    m = t.morb[q, 1].astype(np.int64)
    tz = np.where(req >= t.n_sps, -1, 1)
    M, MT = np.abs(m[:, :3].sum(1)), np.abs(tz[:, :3].sum(1))
    Jmax = np.minimum(j[:, :3].sum(1), j[:, 3:].sum(1))

    def njab(a, b, c, J):
        lo = np.maximum(np.abs(a - b), np.abs(J - c))
        hi = np.minimum(a + b, J + c)
        return np.where(hi >= lo, (hi - lo) // 2 + 1, 0)

    total = np.zeros(len(req), np.int64)
    for J in range(1, int(Jmax.max()) + 1, 2):
        nb = njab(j[:, 0], j[:, 1], j[:, 2], J)
        nk = njab(j[:, 3], j[:, 4], j[:, 5], J)
        live = (J <= Jmax) & (M <= J)
        total += np.where(live & (MT <= 1), nb * nk * 4, 0) + np.where(live, nb * nk, 0)
    return total


def run_threebody(ci, torch, with_oracle, n1max=6, n3max=6):
    """The paper's own GPU kernel: coupled-JT -> m-scheme three-body
    elements on request, timed per chunk of requests (the chunk-size knee)."""
    import seeded_inputs as si

    t = ci.ThreeBody(n1max, n3max)
    A = torch.from_numpy(np.random.default_rng(9).standard_normal(t.n_coupled).astype(np.float32)).cuda()
    req = si.requests_3b(91, 100000, n1max, n3max)
    elems = threebody_block_elements(t, req)
    big = torch.from_numpy(np.ascontiguousarray(np.tile(req, (10, 1)))).cuda()
    out = torch.empty(big.shape[0], dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream()
    rates, ms = {}, {}
    for order in (False, True):
        for n in (1000, 10000, 100000, 1000000):
            r, o = big[:n], out[:n]
            t.decouple(A, r, o, order=order)
            ev = EventTimer(torch, stream)
            for _ in range(5):
                with ev:
                    t.decouple(A, r, o, order=order)
            ms[(order, n)] = ev.mean_ms()
            rates.setdefault("cost_order" if order else "given_order", {})[str(n)] = n / (ms[(order, n)] * 1e-3)
    best = min(ms[(False, 1000000)], ms[(True, 1000000)])
    # algorithmic bytes of one launch of 1e6 requests: the block elements
    # (4 B each), the request (24 B) and the result (4 B)
    alg = 10 * (4 * int(elems.sum()) + 28 * len(req))
    c = measured_counters("decouple_kernel_shells6_n3max6.md")
    res = {"workload": "three-body decoupling, shells 0..%d, triples inside %d, random requests (1e5 distinct)"
           % (n1max, n3max), "n_coupled": t.n_coupled, "requests_per_s_by_chunk": rates,
           "block_elements_per_request": float(elems.mean()),
           "ms_per_launch_1e6": best, "alg_GBps_1e6": alg / (best * 1e-3) / 1e9,
           "roofline": {"bound": "hbm", "achieved": alg / (best * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": alg / (best * 1e-3) / 1e9 / HBM_PEAK_GBS, "alg_bytes_per_launch": alg,
                        "traffic": c.get("traffic_bytes_per_launch") if c else None}}
    if with_oracle:
        # the oracle (plain Python sums) on a sample of the same requests, one core
        from oracle.threebody import ThreeBody as OracleTB

        o3 = OracleTB(n1max, n3max)
        t0 = time.perf_counter()
        k = 0
        while time.perf_counter() - t0 < 5.0 and k < len(req):
            o3.element(req[k], lambda *key: 1.0)
            k += 1
        res.update({"cpu_oracle_requests_per_s": k / (time.perf_counter() - t0), "cpu_oracle_cores": 1,
                    "cpu_oracle_sample": "first %d requests" % k})
    t.free()
    return res


def run_three_body_term(ci, torch, prob, tbme_seed, with_oracle, reps=3):
    """The matrix with a three-body term (states at most three nucleons
    apart, synthetic interaction): count and fill timed with HIP events."""
    import seeded_inputs as si

    b = ci.ci_basis_build([prob])
    stream = torch.cuda.current_stream()
    ev_c, ev_f = EventTimer(torch, stream), EventTimer(torch, stream)
    rp, nnz = ci.ci_hamiltonian3_count(b)
    nnz = nnz[0]
    D = b.info[0]["dim"]
    tb = torch.from_numpy(si.tbme_f32(tbme_seed, b.n_tbme)).cuda()
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    val = torch.empty(nnz, dtype=torch.float32, device="cuda")
    v3 = (ci.CI_V3_SYNTHETIC, 0x5EED3, 1.0)
    ci.ci_hamiltonian3_fill(b, tb, v3, rp, col, val)
    for _ in range(reps):
        with ev_c:
            ci.ci_hamiltonian3_count(b)
        with ev_f:
            ci.ci_hamiltonian3_fill(b, tb, v3, rp, col, val)
    torch.cuda.synchronize()
    fill_ms = ev_f.mean_ms()
    alg = 8 * nnz + 8 * (D + 1)  # col + val per entry, row_ptr per row
    c = measured_counters("h3_rows_fill_li6_nmax6.md")
    res = {"workload": "%s with a three-body term (d <= 3)" % "Z=%d N=%d Nmax=%d 2M=%d" % tuple(prob[:4]),
           "nnz": nnz, "count_ms_incl_sync": ev_c.mean_ms(), "fill_ms": fill_ms,
           "fill_nnz_per_s": nnz / (fill_ms * 1e-3), "fill_alg_GBps": alg / (fill_ms * 1e-3) / 1e9,
           "fill_frac_of_hbm_peak": alg / (fill_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
           "fill_traffic": c.get("traffic_bytes_per_launch") if c else None}
    del col, val
    torch.cuda.empty_cache()
    # the full symmetric matrix with the term, and its lowest eigenpair (Lanczos)
    rpf, nnzf = ci.ci_hamiltonian3_count_full(b)
    colf = torch.empty(nnzf[0], dtype=torch.int32, device="cuda")
    valf = torch.empty(nnzf[0], dtype=torch.float32, device="cuda")
    ci.ci_hamiltonian3_fill_full(b, tb, v3, rpf, colf, valf)
    ev_ff, ev_sp = EventTimer(torch, stream), EventTimer(torch, stream)
    with ev_ff:
        ci.ci_hamiltonian3_fill_full(b, tb, v3, rpf, colf, valf)
    x = torch.ones(D, dtype=torch.float64, device="cuda")
    for _ in range(3):
        with ev_sp:
            y = ci.ci_hamiltonian_spmv(b, 0, rpf, colf, valf, x)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    E, _, it = ci.ci_lanczos(b, 0, rpf, colf, valf, max_iter=300, tol=1e-12)
    t_l = time.perf_counter() - t0
    res.update({"nnz_full": nnzf[0], "fill_full_ms": ev_ff.mean_ms(),
                "spmv_ms": ev_sp.mean_ms(), "spmv_GBps": (8 * nnzf[0] + 24 * D) / (ev_sp.mean_ms() * 1e-3) / 1e9,
                "lanczos_s": t_l, "lanczos_iters": it, "lowest_eigenvalue_MeV": E})
    del colf, valf, y, x
    b.free()
    if with_oracle:
        import oracle

        o = oracle.Oracle(oracle.Problem(*prob))
        o.set_tbme(si.tbme_f32(tbme_seed, o.n_tbme).astype(np.float64))
        o.set_v3(o.V3_SYNTHETIC, 0x5EED3, 1.0)
        rows = si.sample_rows(o.dim, 16, seed=7)
        o.rows3(rows[:2])  # warm-up
        t0 = time.perf_counter()
        counts, _, _ = o.rows3(rows)
        t = time.perf_counter() - t0
        res.update({"cpu_oracle_nnz_per_s": float(counts.sum()) / t, "cpu_oracle_sample": "16 sampled rows",
                    "cpu_oracle_cores": int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))})
    torch.cuda.empty_cache()
    return res


def run_batched(ci, torch, steps, warmup, stored, tuning_text=None):
    """64 bases in one handle; fill + vjp of all of them captured in one HIP
    graph and replayed.  Launch shapes from the library's autotuner."""
    import seeded_inputs as si

    probs, tseeds, pseeds = si.batch_problems()
    t0 = time.perf_counter()
    b = ci.ci_basis_build(probs)
    rp, nnz = ci.ci_hamiltonian_count(b)
    t_setup = time.perf_counter() - t0
    tb = torch.from_numpy(np.concatenate([si.tbme_f32(s, i["n_tbme"]) for s, i in zip(tseeds, b.info)])).cuda()
    tot = int(sum(nnz))
    col = torch.empty(tot, dtype=torch.int32, device="cuda")
    val = torch.empty(tot, dtype=torch.float32, device="cuda")
    G = torch.empty(tot, dtype=torch.float32, device="cuda")
    ci.ci_hamiltonian_fill(b, tb, rp, col, val)
    # upstream psi_i psi_j per basis, built on the device from the structure
    rpc = rp.cpu().numpy()
    for k, i in enumerate(b.info):
        seg = rpc[i["row_ptr_offset"]: i["row_ptr_offset"] + i["dim"] + 1]
        ps = torch.from_numpy(si.psi(pseeds[k], i["dim"])).cuda()
        rows = torch.repeat_interleave(torch.arange(i["dim"], device="cuda"),
                                       torch.from_numpy(np.diff(seg)).cuda())
        G[seg[0]: seg[-1]] = (ps[rows] * ps[col[seg[0]: seg[-1]].long()]).float()
    gt = torch.empty(b.n_tbme, dtype=torch.float32, device="cuda")
    work = torch.empty(max(b.vjp_work_bytes(), 8), dtype=torch.uint8, device="cuda")
    t0 = time.perf_counter()
    if tuning_text:
        b.tuning = parse_tuning(tuning_text)
        tuning = b.tuning
    keys = torch.empty(tot if stored else 0, dtype=torch.int32, device="cuda")
    if not tuning_text:
        tuning = ci.ci_hamiltonian_tune(b, tb, rp, col, val, G, gt, None, reps=2, keys=keys if stored else None)
    t_tune = time.perf_counter() - t0
    work = torch.empty(max(b.vjp_work_bytes(), 8), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()

    def one():
        if stored:
            ci.ci_hamiltonian_fill_keys(b, tb, rp, col, val, keys)
            ci.ci_hamiltonian_vjp_keys(b, rp, keys, G, gt, work)
        else:
            ci.ci_hamiltonian_fill(b, tb, rp, col, val)
            ci.ci_hamiltonian_vjp(b, rp, G, gt, work)

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        for _ in range(2):
            one()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        one()
    for _ in range(warmup):
        g.replay()
    torch.cuda.synchronize()
    a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(steps):
        g.replay()
    e.record()
    torch.cuda.synchronize()
    ms = a.elapsed_time(e) / steps
    dim_total = int(sum(i["dim"] for i in b.info))
    # algorithmic bytes of one replay: fill (8 B per entry + 8 B per row) and
    # adjoint (4 B per entry + 8 B per row + 4 B per table element) of every basis
    alg = 12 * tot + 16 * (dim_total + len(probs)) + 4 * b.n_tbme
    achieved = alg / (ms * 1e-3) / 1e9
    # traffic of one replay: the committed counter summaries of its two kernels
    cf = measured_counters("row_kernel_fill_batch64.md", {k: tuning[k] for k in FILL_SHAPE})
    ca = measured_counters("adjoint_kernel_batch64.md", {k: tuning[k] for k in ADJ_SHAPE})
    traffic = (cf["traffic_bytes_per_launch"] + ca["traffic_bytes_per_launch"]) if (cf and ca and not stored) else None
    out = {"bases": len(probs), "dim_total": dim_total, "nnz_total": tot, "n_tbme_total": b.n_tbme,
           "ms_per_replay": ms, "nnz_per_s": tot / (ms * 1e-3), "setup_s": t_setup,
           "graph": "fill + vjp of all bases, one capture", "adjoint": "stored" if stored else "walk",
           "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": achieved / HBM_PEAK_GBS, "alg_bytes_per_replay": alg, "traffic": traffic},
           "tuning": dict(tuning, tune_s=t_tune, source="fixed" if tuning_text else "autotuner")}
    b.free()
    return out


# VALU wave-instructions/s: a SIMD is 16 lanes wide, so one wave64 VALU
# instruction occupies it for 4 cycles; 256 CUs x 4 SIMDs x 2.4 GHz / 4 =
# 6.14e11/s (= 3.93e13 32-bit lane-ops/s, the published non-packed FP32 rate)
VALU_PEAK = 256 * 4 * 2.4e9 / 4


def leg(ms, nnz, alg_bytes, profile, shape):
    """nonzeros/s, the HBM roofline of the leg's kernel from its algorithmic
    bytes, and the VALU issue fraction from the committed counters of that
    kernel (null when its source changed since they were taken, or when they
    were taken at other launch shapes)."""
    # the kernel's summaries: <profile>.md, and <profile>_<tiles>.md at other launch shapes
    c = None
    for path in sorted(glob.glob(os.path.join(ROOT, "profiles", profile[:-3] + "*.md"))):
        c = measured_counters(os.path.basename(path), shape)
        if c:
            profile = os.path.basename(path)
            break
    achieved = alg_bytes / (ms * 1e-3) / 1e9
    out = {"ms": ms, "nnz_per_s": nnz / (ms * 1e-3),
           "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": achieved / HBM_PEAK_GBS, "alg_bytes_per_launch": alg_bytes,
                        "traffic": c.get("traffic_bytes_per_launch") if c else None,
                        "profile": profile if c else None}}
    insts = c.get("valu_insts_per_launch") if c else None
    out["valu_issue"] = {"insts_per_launch": insts,
                         "frac": insts / (ms * 1e-3) / VALU_PEAK if insts else None,
                         "peak_wave_insts_per_s": VALU_PEAK, "profile": profile if insts else None}
    return out


def parse_tuning(text):
    keys = ("row_waves", "row_grab", "adj_rows", "adj_tile_n", "adj_persistent", "adjk_rows", "adjk_tile_n",
            "adjk_persistent", "row_xcd", "adj_wide", "adj_flush")
    if "=" in text:
        return {k: int(v) for k, v in (kv.split("=") for kv in text.split(","))}
    return dict(zip(keys, (int(x) for x in text.split(","))))


def measure_step(ci, torch, workload, steps, warmup, adjoint, tuning_text):
    """One step = basis build (size query, arena, build, list count, lists) +
    count/scan + fill + adjoint for one problem, inputs (two-body table,
    upstream gradient) resident in HBM.  Returns the timings and legs."""
    import seeded_inputs as si

    w = si.WORKLOADS[workload]
    prob = w["problem"]
    stream = torch.cuda.current_stream()
    # inputs resident in HBM before the timed region: the two-body table and
    # the upstream gradient (which needs the structure, so one setup pass)
    log("setup", workload, prob)
    b = ci.ci_basis_build([prob])
    rp, nnz = ci.ci_hamiltonian_count(b)
    nnz = nnz[0]
    D = b.info[0]["dim"]
    n_tbme = b.n_tbme
    tbme = torch.from_numpy(si.tbme_f32(w["tbme_seed"], n_tbme)).cuda()
    col, val = ci.ci_hamiltonian_fill(b, tbme, rp)
    rows = torch.repeat_interleave(torch.arange(D, device="cuda"), torch.diff(rp))
    ps = torch.from_numpy(si.psi(si.PSI_SEED.get(workload, 0), D)).cuda()
    G = (ps[rows] * ps[col.long()]).float()
    del rows
    gt = torch.empty(n_tbme, dtype=torch.float32, device="cuda")
    work = torch.empty(max(b.vjp_work_bytes(), 8), dtype=torch.uint8, device="cuda")
    # launch shapes picked once by the library's autotuner; the handles built
    # in the timed steps start from them (process-wide cache per problem)
    fixed = None
    t0 = time.perf_counter()
    if tuning_text:
        fixed = parse_tuning(tuning_text)
        b.tuning = fixed
        tuning = b.tuning
    else:
        kt = torch.empty(nnz, dtype=torch.int32, device="cuda") if adjoint == "stored" else None
        tuning = ci.ci_hamiltonian_tune(b, tbme, rp, col, val, G, gt, None, reps=3, keys=kt)
        del kt
    t_tune = time.perf_counter() - t0
    log("launch shapes", tuning, "in %.2f s" % t_tune)
    work = torch.empty(max(b.vjp_work_bytes(), 8), dtype=torch.uint8, device="cuda")
    b.free()
    del col, val
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    val = torch.empty(nnz, dtype=torch.float32, device="cuda")
    stored = adjoint == "stored"
    keys = torch.empty(nnz if stored else 0, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()

    def fill(h, r):
        if stored:
            ci.ci_hamiltonian_fill_keys(h, tbme, r, col, val, keys)
        else:
            ci.ci_hamiltonian_fill(h, tbme, r, col, val)

    def vjp(h, r):
        if stored:
            ci.ci_hamiltonian_vjp_keys(h, r, keys, G, gt, work)
        else:
            ci.ci_hamiltonian_vjp(h, r, G, gt, work)

    t_basis, t_count = [], []
    ev_fill, ev_vjp = EventTimer(torch, stream), EventTimer(torch, stream)

    def step(timed):
        t0 = time.perf_counter()
        h = ci.ci_basis_build([prob])
        if fixed:
            h.tuning = fixed
        t1 = time.perf_counter()
        r, n = ci.ci_hamiltonian_count(h)
        t2 = time.perf_counter()
        if timed:
            t_basis.append(t1 - t0)
            t_count.append(t2 - t1)
            with ev_fill:
                fill(h, r)
            with ev_vjp:
                vjp(h, r)
        else:
            fill(h, r)
            vjp(h, r)
        torch.cuda.synchronize()
        h.free()

    for _ in range(warmup):
        step(False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        step(True)
    torch.cuda.synchronize()
    sec = (time.perf_counter() - t0) / steps
    fill_ms, vjp_ms = ev_fill.mean_ms(), ev_vjp.mean_ms()
    # algorithmic HBM bytes per launch: the fill writes col + val (8 B per
    # stored entry) and reads row_ptr (8 B per row); the adjoint reads the
    # upstream value (4 B per entry) and row_ptr and writes the FP32 table
    # gradient (4 B per table element).  A stored structure word is traffic,
    # not algorithmic bytes.
    fill_alg = 8 * nnz + 8 * (D + 1)
    vjp_alg = 4 * nnz + 8 * (D + 1) + 4 * n_tbme
    fwd = leg(fill_ms, nnz, fill_alg, ("row_kernel_fill_keys_%s.md" if stored else "row_kernel_fill_%s.md")
              % workload, {k: tuning[k] for k in FILL_SHAPE})
    adj = leg(vjp_ms, nnz, vjp_alg, ("adjoint_stored_kernel_%s.md" if stored else "adjoint_kernel_%s.md")
              % workload, {k: tuning[k] for k in (ADJK_SHAPE if stored else ADJ_SHAPE)})
    return {"prob": prob, "dim": D, "nnz": nnz, "n_tbme": n_tbme, "sec": sec, "tuning": tuning,
            "tune_s": t_tune, "fixed": fixed is not None,
            "stages_ms": {"basis_build": 1e3 * float(np.mean(t_basis)),
                          "count_scan_sync": 1e3 * float(np.mean(t_count)), "fill": fill_ms, "vjp": vjp_ms},
            "fwd": fwd, "adjoint": adj, "adjoint_kind": "stored structure words" if stored else
            "recomputed structure (partner-list walk)"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="b10_nmax4",
                    help="headline workload: b10_nmax4 (Z=5, N=5, Nmax=4, 2M=0: forward + adjoint) by default")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-batched", action="store_true")
    ap.add_argument("--only-threebody", action="store_true",
                    help="run only the three-body decoupling section (for counter and trace runs of its kernels)")
    ap.add_argument("--only-three-body-term", action="store_true",
                    help="run only the section of the matrix with a three-body term (counter and trace runs)")
    ap.add_argument("--only-step", action="store_true",
                    help="run only the timed construction steps of the headline workload (for counter and "
                         "trace runs of the step's kernels)")
    ap.add_argument("--only-batched", action="store_true",
                    help="run only the batched section (for counter and trace runs of its kernels)")
    ap.add_argument("--tuning", default=None, metavar="SHAPES",
                    help="fixed launch shapes instead of the autotuner (for profiling runs): "
                         "row_waves,row_grab,adj_rows,adj_tile_n,adj_persistent[,adjk_rows,adjk_tile_n] "
                         "or name=value pairs")
    ap.add_argument("--adjoint", choices=("walk", "stored"), default="walk",
                    help="walk (default): the adjoint recomputes the pair and phase structure by walking the "
                         "partner lists; stored: the fill stores one structure word per entry and the adjoint "
                         "reads them")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="after the timed steps, copy MIB MiB device to device three times (a plain "
                         "copy of known size, to scale hardware byte counters under rocprofv3)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU only: the construction path here runs on a single "
              "MI355X (multi-GPU sharding is described in the design notes, not run).", file=sys.stderr)
        sys.exit(2)

    import torch

    import seeded_inputs as si

    ci = ensure_library()
    if args.only_threebody:
        res = {"threebody": run_threebody(ci, torch, not args.no_cpu_baseline)}
        copy_calibration(torch, args.copy_calibration)
        print(json.dumps(res), flush=True)
        return
    w = si.WORKLOADS[args.workload]
    prob = w["problem"]
    if args.only_three_body_term:
        res = {"three_body_term": run_three_body_term(ci, torch, prob, w["tbme_seed"], not args.no_cpu_baseline)}
        copy_calibration(torch, args.copy_calibration)
        print(json.dumps(res), flush=True)
        return
    if args.only_batched:
        res = {"batched": run_batched(ci, torch, max(2, args.steps), args.warmup, args.adjoint == "stored",
                                      args.tuning)}
        copy_calibration(torch, args.copy_calibration)
        print(json.dumps(res), flush=True)
        return

    m = measure_step(ci, torch, args.workload, args.steps, args.warmup, args.adjoint, args.tuning)
    copy_calibration(torch, args.copy_calibration)
    nnz, D = m["nnz"], m["dim"]
    dom = "fwd" if m["fwd"]["ms"] >= m["adjoint"]["ms"] else "adjoint"
    r = m[dom]["roofline"]
    res = {
        "metric": "Hamiltonian nonzeros/sec (fwd, adjoint, batched) + roofline fraction, 1 MI355X",
        "value": nnz / m["sec"],
        "unit": "nonzeros/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": m["sec"] * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int32+f32 (f64 sums in the fill, int64 fixed-point sums in the adjoint)",
        "data": "synthetic: seeded N(0,1) MeV two-body table, seeded psi for the upstream gradient",
        "config": {"workload": args.workload, "Z": prob[0], "N": prob[1], "nmax": prob[2],
                   "two_m": prob[3], "parity": prob[4], "dim": D, "nnz": nnz, "n_tbme": m["n_tbme"],
                   "step": "basis build + count/scan + fill + adjoint (vjp)", "adjoint": m["adjoint_kind"]},
        "stages_ms": m["stages_ms"],
        "tuning": dict(m["tuning"], tune_s=m["tune_s"], source="fixed" if m["fixed"] else "autotuner"),
        "fwd": m["fwd"],
        "adjoint": m["adjoint"],
        "roofline": {"kernel": "fill" if dom == "fwd" else "vjp", "bound": "hbm", "achieved": r["achieved"],
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": r["frac"], "traffic": r["traffic"],
                     "alg_bytes_per_launch": r["alg_bytes_per_launch"]},
    }
    if args.only_step:
        print(json.dumps(res), flush=True)
        return
    # the 6Li Nmax=6 workload (W = 4 words per species, 3.97e6 table elements)
    log("li6")
    m6 = measure_step(ci, torch, "li6_nmax6", max(3, args.steps // 2), 1, args.adjoint, None)
    res["li6_nmax6"] = {"dim": m6["dim"], "nnz": m6["nnz"], "n_tbme": m6["n_tbme"],
                        "step_nnz_per_s": m6["nnz"] / m6["sec"], "ms_per_step": m6["sec"] * 1e3,
                        "stages_ms": m6["stages_ms"], "fwd": m6["fwd"], "adjoint": m6["adjoint"],
                        "tuning": m6["tuning"]}
    # measured machine ceilings (streaming stores; XOR + popcount issue rate)
    ceil = ci.ci_probe_ceilings(1024)
    res["measured_ceilings"] = {
        "store_GBps": ceil["store_GBps"],
        "xor_popcount_steps_per_s": ceil["xor_popcount_steps_per_s"],
        "valu_lane_ops_per_s": 5 * ceil["xor_popcount_steps_per_s"],
        "fill_frac_of_measured_store": m["fwd"]["roofline"]["achieved"] / ceil["store_GBps"],
    }
    if not args.no_batched:
        log("batched")
        res["batched"] = run_batched(ci, torch, max(3, args.steps // 2), 1, args.adjoint == "stored", None)
    log("lanczos")
    res["lanczos"] = run_lanczos(ci, torch, si.WORKLOADS["li6_nmax6"]["problem"], si.WORKLOADS["li6_nmax6"]["tbme_seed"])
    log("three-body")
    res["threebody"] = run_threebody(ci, torch, not args.no_cpu_baseline)
    log("three-body term")
    res["three_body_term"] = run_three_body_term(ci, torch, si.WORKLOADS["li6_nmax6"]["problem"],
                                                 si.WORKLOADS["li6_nmax6"]["tbme_seed"], not args.no_cpu_baseline)
    if not args.no_cpu_baseline:
        log("cpu baseline")
        res["cpu_baseline"] = cpu_baseline(prob, w["tbme_seed"], si.PSI_SEED.get(args.workload, 0))
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
