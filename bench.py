"""Benchmark of the MDF-LBM hot path on one MI355X.

Workload (the largest configuration that fits one GPU): 512 seeded,
independent 2D cases of uneven size (lid-driven cavities and body-force
channels, N x N with N in {64, 96, ..., 512}, Re log-uniform in [10, 1000],
lid or centreline speed in [0.05, 0.1]; 53.6 M nodes), D2Q5 with three
distribution sets (ubar_0, u, v), FP64 storage (the paper's arithmetic),
halfway anti-bounce-back walls; all cases advance together in batched
launches of one step, or of several where the autotuner picks that form, and every 100 steps the FP64 K-interval
residual of every case is evaluated inside the last step of the chunk and
read back (the loop of a steady solve).  A step is one pass of all of that
over every case.

Prints one JSON line: MLUPS (whole job), the roofline of the dominant
kernel (algorithmic bytes per launch over the HIP-event-timed average
launch duration, against 8 TB/s), the FP32 cavity kernels on 1024^2 and
8192^2 grids as extra entries, and the FP64 CPU oracle timed on a bounded
sample of the same cases.
"""
import argparse
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0


def kernel_source_hash():
    """Hash of what determines the step kernels' machine code: their sources
    and the compiler flags."""
    from paper_2108_08591_amd import build as B
    h = hashlib.sha256()
    for name in B.KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2108_08591_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    h.update(" ".join(B.HIP_FLAGS).encode())
    return h.hexdigest()[:16]


def measured_traffic(kernel_key, launches_bytes):
    """HBM bytes per launch from the committed rocprofv3 counter summary, or
    None when the kernel source changed since the counters were taken."""
    path = os.path.join(ROOT, "profiles", "traffic_counters.json")
    if not os.path.exists(path):
        return None
    try:
        data = json.load(open(path))
    except (OSError, ValueError):
        return None
    ent = data.get(kernel_key)
    if not ent or ent.get("source_hash") != kernel_source_hash():
        return None
    return ent.get("bytes_per_launch")


def device_copy_bandwidth(nbytes=1 << 30, reps=5):
    """Context for the roofline: a plain device-to-device copy of `nbytes`
    (torch copy_, one read and one write per byte), HIP events, best of reps."""
    import torch
    a = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    b = torch.empty_like(a)
    a.fill_(1)
    b.copy_(a)
    best = None
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        b.copy_(a)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1)
        best = ms if best is None else min(best, ms)
    del a, b
    torch.cuda.empty_cache()
    return {"GBps": round(2 * nbytes / (best / 1e3) / 1e9, 1), "bytes_copied": nbytes,
            "kind": "torch copy_ device to device, read + write bytes, HIP events, best of %d" % reps}


def cpu_baseline_batch(target_s=15.0, steps=40):
    """The FP64 oracle as it stands, timed on a bounded sample of the same
    workload: the cases of the seeded 512-case batch in their seeded order,
    `steps` steps each (collide + stream), until about target_s seconds of
    CPU work; MLUPS over the cases run."""
    import numpy as np
    from oracle import oracle as O
    from paper_2108_08591_amd import cases as C

    done_nodes, el, names = 0, 0.0, []
    for bc in C.batch_cases(n=512):
        sp = bc.spec
        o = O.Oracle(O.Case(sp.lattice, sp.shape, sp.s1, bc=sp.bc, wall_u=sp.wall_velocity(), force=sp.force))
        o.init(0.0, np.zeros((2,) + sp.fshape))
        t0 = time.perf_counter()
        o.run(steps)
        el += time.perf_counter() - t0
        done_nodes += sp.nodes * steps
        names.append(f"{bc.kind} {bc.N}^2")
        if el >= target_s:
            break
    threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    return {
        "value": round(done_nodes / el / 1e6, 3),
        "unit": "MLUPS",
        "cores": threads,
        "kind": "oracle",
        "sample": f"FP64 oracle on the first {len(names)} cases of the same seeded 512-case batch "
                  f"({', '.join(names)}), {steps} steps each from rest",
        "seconds": round(el, 2),
    }


def copy_calibration():
    """A plain device-to-device copy of known size (256 MiB read + 256 MiB
    written per launch, beyond the Infinity Cache), run under the HBM traffic
    counters to calibrate them."""
    import torch
    n = 64 * 1024 * 1024
    a = torch.ones(n, dtype=torch.float32, device="cuda:0")
    b = torch.empty_like(a)
    for _ in range(10):
        b.copy_(a)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record()
    for _ in range(20):
        b.copy_(a)
    ev1.record()
    torch.cuda.synchronize()
    ms = ev0.elapsed_time(ev1) / 20
    print(json.dumps({"copy_bytes_per_launch": 2 * 4 * n, "copy_ms": round(ms, 4),
                      "copy_GBps": round(2 * 4 * n / (ms / 1e3) / 1e9, 1)}), flush=True)


def _short_kernel_name(name):
    base = name[5:] if name.startswith("void ") else name
    base = base.replace("(anonymous namespace)::", "").replace("mdf::", "")
    return base.split("(")[0]


def summarize_trace(db_path, command):
    """Markdown summary of a rocprofv3 --kernel-trace --stats database, one
    row per kernel and grid size."""
    import sqlite3
    cur = sqlite3.connect(db_path).cursor()
    rows = list(cur.execute(
        "select name, grid_x * grid_y * grid_z as g, count(*), sum(duration) / 1000.0, "
        "avg(duration) / 1000.0 from kernels group by name, g order by sum(duration) desc"))
    total = sum(r[3] for r in rows)
    out = ["# rocprofv3 kernel trace", "", "Command (run from the repository root on an MI355X):", "",
           "```", command, "```", "",
           "| kernel | grid (work-items) | calls | total (us) | average (us) | % |", "|---|---|---|---|---|---|"]
    for name, g, calls, tot, avg in rows:
        out.append(f"| `{_short_kernel_name(name)}` | {g} | {calls} | {tot:.1f} | {avg:.3f} | "
                   f"{100.0 * tot / total:.2f} |")
    return "\n".join(out) + "\n"


def counter_means(db_path, counter):
    """Mean of a counter per (kernel, grid size): {(name, grid): (dispatches, mean)}."""
    import sqlite3
    import statistics
    cur = sqlite3.connect(db_path).cursor()
    acc = {}
    for name, g, val in cur.execute("select kernel_name, grid_size, value from counters_collection "
                                    "where counter_name=?", (counter,)):
        acc.setdefault((_short_kernel_name(name), g), []).append(val)
    return {k: (len(v), statistics.mean(v)) for k, v in acc.items()}


def summarize_traffic(fetch_db, write_db, copy_fetch_db, copy_write_db, kernel_prefix, alg_bytes,
                      kernel_key, commands):
    """Calibrated HBM bytes per launch of one kernel from FETCH_SIZE and
    WRITE_SIZE runs (KiB per dispatch), each scaled by what the same counter
    reads for a plain copy of known size."""
    f = counter_means(fetch_db, "FETCH_SIZE")
    w = counter_means(write_db, "WRITE_SIZE")
    cf = counter_means(copy_fetch_db, "FETCH_SIZE")
    cw = counter_means(copy_write_db, "WRITE_SIZE")
    copy_kib = 256 * 1024
    ck = [k for k in cf if "copyBuffer" in k[0]][0]
    fetch_scale = copy_kib / cf[ck][1]
    write_scale = copy_kib / cw[ck][1]
    # the step kernel on the benchmark grid: the most frequent dispatch shape
    kf = max((k for k in f if k[0].startswith(kernel_prefix)), key=lambda k: f[k][0])
    kw = max((k for k in w if k[0].startswith(kernel_prefix)), key=lambda k: w[k][0])
    fetch_b = f[kf][1] * 1024 * fetch_scale
    write_b = w[kw][1] * 1024 * write_scale
    total = fetch_b + write_b
    md = ["# HBM traffic of `" + kernel_prefix + "`", "", "Commands (repository root, on an MI355X):", "", "```"]
    md += commands + ["```", "",
                      f"* copy calibration (256 MiB read + 256 MiB written per launch): FETCH_SIZE reads "
                      f"{cf[ck][1]:.1f} KiB (scale {fetch_scale:.4f}), WRITE_SIZE reads {cw[ck][1]:.1f} KiB "
                      f"(scale {write_scale:.4f})",
                      f"* kernel: FETCH_SIZE {f[kf][1]:.1f} KiB over {f[kf][0]} dispatches, WRITE_SIZE "
                      f"{w[kw][1]:.1f} KiB over {w[kw][0]} dispatches",
                      f"* calibrated bytes per launch: read {fetch_b / 1e6:.2f} MB + write {write_b / 1e6:.2f} MB "
                      f"= {total / 1e6:.2f} MB; algorithmic {alg_bytes / 1e6:.2f} MB "
                      f"(ratio {total / alg_bytes:.3f})", ""]
    ent = {"bytes_per_launch": round(total), "read_bytes": round(fetch_b), "write_bytes": round(write_b),
           "algorithmic_bytes": alg_bytes, "fetch_scale": fetch_scale, "write_scale": write_scale,
           "source_hash": kernel_source_hash()}
    return "\n".join(md) + "\n", {kernel_key: ent}


def parse_launch(text):
    """'128x2g8t' -> (128, 2, 8, 2): tile of 128 x 2 threads, 8 XCD bands and
    the step-kernel form: 's' one node per thread (default, 0), 'v' vector
    (1), 't' several steps per launch (2)."""
    t = text.lower()
    form = 0
    if t[-1] in "svt":
        form = "svt".index(t[-1])
        t = t[:-1]
    groups = 1
    if "g" in t:
        t, g = t.split("g")
        groups = int(g)
    bx, by = (int(v) for v in t.split("x"))
    return bx, by, groups, form


def time_launches(solver, stream, n, fields=0, out=None, reps=3):
    """Average duration of one step-kernel launch (HIP events around n
    back-to-back launches on the kernel's stream, median of reps), in ms."""
    import statistics
    import torch
    res = []
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        if fields:
            solver.step_emit(n, fields, out)
        else:
            solver.step(n)
        e1.record(stream)
        torch.cuda.synchronize()
        res.append(e0.elapsed_time(e1) / n)
    return statistics.median(res)


def variants_study(out_path):
    """Cost of each variant of the update against the plain one on the same
    grid, storage and default launch shape (several steps per launch on the 2D
    axis-link lattices, one node per thread elsewhere),
    stepping without field emission: the d velocity sets only (Remark IV),
    Scheme II forcing (eq. 2-3c), and a per-node force field (d more reads
    per node and step).  Algorithmic bytes per step: one read and one write
    of every stored population, plus the force field when one is set."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    sb = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}
    cb = {"f64": 8, "f32": 4, "f16dev": 4, "bf16dev": 4}       # compute dtype of the force field
    names = {C.D2Q5: "d2q5", C.D3Q7: "d3q7", C.D2Q4: "d2q4", C.D3Q6: "d3q6", C.D2Q9: "d2q9", C.D3Q15: "d3q15"}
    runs = [(C.D2Q5, 1024, "f32"), (C.D2Q5, 8192, "f32"), (C.D2Q5, 8192, "f16dev"), (C.D2Q5, 8192, "f64"),
            (C.D3Q7, 256, "f32"), (C.D3Q7, 256, "f16dev"), (C.D3Q7, 256, "f64"),
            (C.D2Q4, 8192, "f32"), (C.D2Q4, 8192, "f16dev"), (C.D3Q6, 256, "f32"), (C.D3Q6, 256, "f16dev"),
            (C.D2Q9, 8192, "f32"), (C.D3Q15, 256, "f32")]
    variants = [("all", C.PLAIN, False), ("velocity", C.PLAIN, False), ("all", C.SCHEME2, False),
                ("all", C.PLAIN, True), ("velocity", C.SCHEME2, True)]
    with open(out_path, "w") as fh:
        for lid, N, st in runs:
            lat = names[lid]
            if C.DIM[lid] == 2:
                spec = C.cavity_case(N=N, Re=1000.0, lattice=lid)
            else:
                spec = C.tgv3d_case(N=N, u0=0.05, Re=100.0, lattice=lid)
            q = spec.q
            base = None
            for sets, forcing, field in variants:
                spec.forcing = forcing
                solver = mdf.Solver([spec], storage=st, device=dev, stream=stream, u_ref=0.1, sets=sets)
                if field:
                    ff = torch.full((spec.d,) + spec.fshape, 1e-7, dtype=solver.dtype, device=dev)
                    solver.set_force_field(ff)
                solver.step(3)
                ms = time_launches(solver, stream, 41)
                step_bytes = spec.nodes * (2 * q * solver.nsets * sb[st] + (spec.d * cb[st] if field else 0))
                rec = {"lattice": lat, "N": N, "storage": st, "sets": sets,
                       "forcing": "scheme2" if forcing == C.SCHEME2 else "plain", "force_field": field,
                       "ms_per_step": round(ms, 5), "MLUPS": round(spec.nodes / ms / 1e3, 1),
                       "step_bytes_MB": round(step_bytes / 1e6, 1),
                       "GBps_per_step": round(step_bytes / ms / 1e6, 1)}
                if base is None:
                    base = ms
                else:
                    rec["speedup_vs_plain_all_sets"] = round(base / ms, 3)
                print(json.dumps(rec), file=fh, flush=True)
                print(json.dumps(rec), flush=True)
                del solver
                torch.cuda.empty_cache()


def lattice_per_set_study(out_path):
    """A lattice per set against the plain diagonal lattice on the same grid:
    D2Q9 at 8192^2 and D3Q15 at 256^3, all d + 1 sets on the large lattice,
    the set a = 0 on D2Q5 / D3Q7 (23 and 52 planes per buffer instead of 27
    and 60), and the velocity sets only; one node per thread, no emission.
    Algorithmic bytes per step: one read and one write of every stored
    population."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    sb = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}
    runs = [(2, 8192, "f32"), (2, 8192, "f64"), (3, 256, "f32"), (3, 256, "f64")]
    with open(out_path, "w") as fh:
        for d, N, st in runs:
            big, mixed = (C.D2Q9, C.D2Q9_Q5) if d == 2 else (C.D3Q15, C.D3Q15_Q7)
            base = None
            for lid, sets, label in ((big, "all", "large lattice, d+1 sets"),
                                     (mixed, "all", "lattice per set"),
                                     (big, "velocity", "large lattice, velocity sets")):
                if d == 2:
                    spec = C.cavity_case(N=N, Re=1000.0, lattice=lid)
                else:
                    spec = C.tgv3d_case(N=N, u0=0.05, Re=100.0, lattice=lid)
                solver = mdf.Solver([spec], storage=st, device=dev, stream=stream, sets=sets)
                solver.step(3)
                ms = time_launches(solver, stream, 41)
                q = spec.q
                planes = (2 * d + 1 + d * q) if lid == mixed else solver.nsets * q
                step_bytes = spec.nodes * 2 * planes * sb[st]
                rec = {"lattice": label, "lattice_id": lid, "d": d, "N": N, "storage": st, "planes": planes,
                       "ms_per_step": round(ms, 5), "MLUPS": round(spec.nodes / ms / 1e3, 1),
                       "step_bytes_MB": round(step_bytes / 1e6, 1),
                       "GBps_per_step": round(step_bytes / ms / 1e6, 1),
                       "roofline_frac": round(step_bytes / ms / 1e6 / HBM_PEAK_GBS, 4)}
                if base is None:
                    base = ms
                else:
                    rec["speedup_vs_large_lattice"] = round(base / ms, 3)
                print(json.dumps(rec), file=fh, flush=True)
                print(json.dumps(rec), flush=True)
                del solver
                torch.cuda.empty_cache()


BF16_DENSE_PEAK_TFLOPS = 2500.0      # MI355X dense BF16 matrix peak (no sparsity)


def conv_study(out_path, B=16, N=256, reps=5):
    """The warm-start network's 3x3 convolutions at the configured image size
    (N^2, batch B), layer by layer: forward, data gradient (forward with the
    flipped weights, cout <-> cin) and weight gradient, each timed with HIP
    events (median of reps) and priced at 2 * pixels * cout * 9 * cin flops
    against the dense BF16 matrix peak."""
    import torch
    from paper_2108_08591_amd import nn
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    g = torch.Generator(device="cpu").manual_seed(7)
    layers = []
    H = N
    cin = nn.IN_CH
    for l, c in enumerate(nn.LEVELS):
        layers.append((f"enc{l}a", H, cin, 0, c))
        layers.append((f"enc{l}b", H, c, 0, c))
        cin = c
        if l < len(nn.LEVELS) - 1:
            H //= 2
    for l in range(len(nn.LEVELS) - 2, -1, -1):
        H *= 2
        c = nn.LEVELS[l]
        layers.append((f"dec{l}a", H, nn.LEVELS[l + 1], c, c))
        layers.append((f"dec{l}b", H, c, 0, c))

    def rnd(*shape):
        return nn.to_bf16((torch.randn(*shape, generator=g) * 0.1).to(dev))

    def timed(fn):
        ts = []
        for _ in range(reps):
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            with torch.cuda.stream(stream):
                e0.record(stream)
                fn()
                e1.record(stream)
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        return sorted(ts)[len(ts) // 2]

    recs = []
    with open(out_path, "w") as fh:
        for name, HH, c1, c2, co in layers:
            x1 = rnd(B, HH, HH, c1)
            x2 = rnd(B, HH, HH, c2) if c2 else None
            w = rnd(co, 9, c1 + c2)
            bias = torch.zeros(co, device=dev)
            y = nn.bf16_empty((B, HH, HH, co), dev)
            dy = rnd(B, HH, HH, co)
            dx = nn.bf16_empty((B, HH, HH, c1), dev)
            wt = nn.bf16_empty((c1 + c2, 9, co), dev)
            dw = torch.zeros(co, 9, c1 + c2, device=dev)
            db = torch.zeros(co, device=dev)
            scratch = torch.empty(nn.wgrad_scratch_bytes(B, HH, HH, c1 + c2, co), dtype=torch.uint8, device=dev)
            nn.conv_flip(w, wt, stream)
            flops = 2.0 * B * HH * HH * co * 9 * (c1 + c2)
            fwd = lambda: nn.conv_fwd(x1, x2, w, bias, True, out_bf16=y, stream=stream)
            dgrad = lambda: nn.conv_fwd(dy, None, wt[:c1], None, False, out_bf16=dx, stream=stream)
            wgrad = lambda: nn.conv_wgrad(x1, x2, dy, dw, db, scratch, stream)
            for kind, fn, fl in (("fwd", fwd, flops), ("dgrad", dgrad, 2.0 * B * HH * HH * c1 * 9 * co),
                                 ("wgrad", wgrad, flops)):
                fn()
                ms = timed(fn)
                tf = fl / ms / 1e9
                rec = {"layer": name, "kind": kind, "B": B, "H": HH, "cin": c1 + c2, "cout": co,
                       "ms": round(ms, 4), "GFLOP": round(fl / 1e9, 2), "TFLOPs": round(tf, 1),
                       "frac_bf16_peak": round(tf / BF16_DENSE_PEAK_TFLOPS, 4)}
                recs.append(rec)
                print(json.dumps(rec), file=fh, flush=True)
                print(json.dumps(rec), flush=True)
            del x1, x2, w, y, dy, dx, wt, dw, scratch
            torch.cuda.empty_cache()
        tot_ms = sum(r["ms"] for r in recs)
        tot_fl = sum(r["GFLOP"] for r in recs)
        summ = {"summary": "one training step's convolutions", "B": B, "N": N, "ms": round(tot_ms, 3),
                "GFLOP": round(tot_fl, 1), "TFLOPs": round(tot_fl / tot_ms, 1),
                "frac_bf16_peak": round(tot_fl / tot_ms / BF16_DENSE_PEAK_TFLOPS, 4)}
        print(json.dumps(summ), file=fh, flush=True)
        print(json.dumps(summ), flush=True)


def sweep(out_path):
    """Step-kernel timing over grid sizes (incl. working sets far beyond the
    256 MB Infinity Cache), storages, lattices and launch shapes."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    sb = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}
    runs = []
    for N in (1024, 2048, 4096, 8192):
        for st in ("f32", "f64", "f16dev", "bf16dev"):
            runs.append(("d2q5", N, st))
    for N in (128, 256, 384):
        for st in ("f32", "f64", "f16dev", "bf16dev"):
            runs.append(("d3q7", N, st))
    shapes = [(64, 4, 8, 1), (128, 2, 8, 1), (256, 1, 8, 1), (64, 2, 8, 1), (128, 2, 1, 1), (64, 4, 8, 0),
              (128, 2, 8, 0), (256, 1, 8, 0), (64, 4, 1, 0), (128, 2, 1, 0), (128, 2, 8, 2), (128, 2, 1, 2)]
    with open(out_path, "w") as fh:
        for lat, N, st in runs:
            if lat == "d2q5":
                spec = C.cavity_case(N=N, Re=1000.0)
                q, ns = 5, 3
            else:
                spec = C.tgv3d_case(N=N, u0=0.05, Re=100.0)
                q, ns = 7, 4
            try:
                solver = mdf.Solver([spec], storage=st, device=dev, stream=stream, u_ref=0.1)
            except Exception as e:           # out of memory on the largest grids
                print(json.dumps({"lattice": lat, "N": N, "storage": st, "error": str(e)[:100]}), file=fh)
                continue
            nodes = spec.nodes
            alg = nodes * 2 * q * ns * sb[st]
            n = max(5, min(400, int(2e10 / alg)))
            for bx, by, g, form in shapes:
                solver.set_launch(bx, by, g, form)
                solver.step(2)
                ms = time_launches(solver, stream, n)
                rec = {"lattice": lat, "N": N, "storage": st, "launch": f"{bx}x{by}g{g}{'svt'[form]}",
                       "ms": round(ms, 5), "MLUPS": round(nodes / ms / 1e3, 1),
                       "GBps": round(alg / ms / 1e6, 1), "frac": round(alg / ms / 1e6 / HBM_PEAK_GBS, 4),
                       "working_set_MB": round(2 * alg / 2 / 1e6, 1)}
                print(json.dumps(rec), file=fh, flush=True)
                print(json.dumps(rec), flush=True)
            del solver
            torch.cuda.empty_cache()


def tgv3d_timing(storage, form, N=256, groups=8, quiet=False, bx=64, by=4, tune=False):
    """The 3D Taylor-Green vortex of the precision configuration (D3Q7, four
    sets, Re 100, u0 = 0.05) at N^3: time per step of the step kernel in one
    storage and form on bx x by threads per block (tune: the form and
    shape mdf_autotune picks instead), HIP events, median of 5, and its
    per-step fraction of the HBM roofline (2 x 28 values per node and
    step).  Returns the record (and prints it unless quiet)."""
    import numpy as np
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    spec = C.tgv3d_case(N=N, u0=0.05, Re=100.0)
    P, u = C.taylor_green_3d_initial(N, 0.05)
    dt = np.float64 if storage == "f64" else np.float32
    init = torch.tensor(np.concatenate([P[None], u]).astype(dt))
    del P, u
    solver = mdf.Solver([spec], storage=storage, init=("fields", [init]), device=dev, stream=stream, u_ref=0.05)
    del init
    if tune:
        bx, by, groups, form = solver.autotune(trial_steps=20)[0]
    else:
        solver.set_launch(bx, by, groups, form)
    solver.step(3)
    n = 41 if form == 2 else 40
    ms = time_launches(solver, stream, n, reps=5)
    sb = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}[storage]
    mlups = spec.nodes / ms / 1e3
    rec = {"workload": f"3D Taylor-Green {N}^3, D3Q7 x 4 sets", "storage": storage, "form": form,
           "groups": groups, "block": f"{bx}x{by}", "ms_per_step": round(ms, 5), "MLUPS": round(mlups, 1),
           "per_step_frac": round(mlups * 1e6 * 2 * 28 * sb / (HBM_PEAK_GBS * 1e9), 4)}
    del solver
    torch.cuda.empty_cache()
    if not quiet:
        print(json.dumps(rec), flush=True)
    return rec


def grid2d_timing(storage, form, N=8192, groups=8, quiet=False):
    """The lid-driven cavity of the channel-and-cavity configuration (D2Q5,
    three sets, Re 1000, lid 0.1) at N^2 without field emission: time per
    step of the step kernel in one storage and form, HIP events, median of
    5, and its per-step fraction of the HBM roofline (2 x 15 values per node
    and step).  Returns the record (and prints it unless quiet)."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    spec = C.cavity_case(N=N, Re=1000.0, U=0.1)
    solver = mdf.Solver([spec], storage=storage, device=dev, stream=stream, u_ref=0.1)
    solver.set_launch(64, 4, groups, form)
    solver.step(3)
    n = 41 if form == 2 else 40
    ms = time_launches(solver, stream, n, reps=5)
    sb = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}[storage]
    mlups = spec.nodes / ms / 1e3
    rec = {"workload": f"lid-driven cavity {N}^2, D2Q5 x 3 sets", "storage": storage, "form": form,
           "groups": groups, "ms_per_step": round(ms, 5), "MLUPS": round(mlups, 1),
           "per_step_frac": round(mlups * 1e6 * 2 * 15 * sb / (HBM_PEAK_GBS * 1e9), 4)}
    del solver
    torch.cuda.empty_cache()
    if not quiet:
        print(json.dumps(rec), flush=True)
    return rec


def summarize_counters(db_paths, command, node_steps, kernel_prefix):
    """Markdown summary of rocprofv3 --pmc runs for one kernel: the mean of
    every counter per dispatch of the most frequent dispatch shape, and the
    per-node-step figures the instruction counters give (SQ_INSTS_* count
    wave instructions; one wave covers 64 node-steps of a one-node-per-thread
    kernel, so per node-step = count x 64 / node_steps)."""
    import sqlite3
    import statistics
    rows = {}
    for db in db_paths:
        cur = sqlite3.connect(db).cursor()
        acc = {}
        for name, g, cname, val in cur.execute("select kernel_name, grid_size, counter_name, value "
                                               "from counters_collection"):
            k = _short_kernel_name(name)
            if not k.startswith(kernel_prefix):
                continue
            acc.setdefault((k, g, cname), []).append(val)
        for (k, g, cname), v in acc.items():
            rows.setdefault(cname, []).append((len(v), statistics.mean(v), k, g))
    out = ["# rocprofv3 counters of `" + kernel_prefix + "`", "", "Commands (repository root, on an MI355X):", "",
           "```"] + command.split(" ;; ") + ["```", "",
           f"Node-steps per dispatch: {node_steps}.", "",
           "| counter | dispatches | mean per dispatch | per node-step |", "|---|---|---|---|"]
    vals = {}
    for cname in sorted(rows):
        n, mean, k, g = max(rows[cname])
        vals[cname] = mean
        per = ""
        if cname.startswith("SQ_INSTS_"):
            per = f"{mean * 64 / node_steps:.1f}"
        out.append(f"| {cname} | {n} | {mean:.4g} | {per} |")
    out.append("")
    if "GRBM_GUI_ACTIVE" in vals:
        # GRBM_GUI_ACTIVE is summed over the 8 XCDs
        cyc = vals["GRBM_GUI_ACTIVE"] / 8
        out.append(f"* duration: {cyc:.0f} GPU cycles per dispatch (GRBM_GUI_ACTIVE / 8 XCDs)")
        if "SQ_INSTS_VALU" in vals:
            # a CU issues at most one wave64 VALU instruction per cycle (four
            # SIMDs, four cycles each, no packed FP32)
            out.append(f"* VALU issue: SQ_INSTS_VALU / (256 CUs x cycles) = "
                       f"{vals['SQ_INSTS_VALU'] / (256 * cyc):.3f}")
    if "SQ_WAVE_CYCLES" in vals and "SQ_WAVES" in vals:
        out.append(f"* mean wave lifetime: SQ_WAVE_CYCLES / SQ_WAVES = {vals['SQ_WAVE_CYCLES'] / vals['SQ_WAVES']:.0f}")
    if "SQ_WAIT_INST_ANY" in vals and "SQ_WAVE_CYCLES" in vals:
        out.append(f"* SQ_WAIT_INST_ANY / SQ_WAVE_CYCLES = {vals['SQ_WAIT_INST_ANY'] / vals['SQ_WAVE_CYCLES']:.3f}")
    return "\n".join(out) + "\n"


def _rel(ref, got, scale=None):
    import torch
    num = torch.linalg.vector_norm((ref - got.to(ref.dtype)).reshape(-1)).item()
    den = torch.linalg.vector_norm(ref.reshape(-1)).item()
    if scale is not None:
        den = max(den, scale)
    return num / den if den > 0 else num


def precision_study(out_path, N=256, steps=(1000, 2500, 5000)):
    """3D Taylor-Green on a periodic N^3 box, D3Q7 x 4 sets, u0 = 0.05,
    Re = 100 and 1600: FP32, FP16- and BF16-deviation storage against the
    FP64-storage run of the same kernels (whose parity with the FP64 oracle
    is tested at small sizes), relative L2 error per field at each step
    count, and the step time of each storage."""
    import numpy as np
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    fields = mdf.FIELD_MOMENTS | mdf.FIELD_VORT
    res = []
    P, u = C.taylor_green_3d_initial(N, 0.05)
    init64 = torch.tensor(np.concatenate([P[None], u], axis=0))
    del P, u
    for Re in (100.0, 1600.0):
        spec = C.tgv3d_case(N=N, u0=0.05, Re=Re)
        if Re > 1000.0:
            # s1 = 1.98 here; the even-moment rate 8(2-s1)/(8-s1) = 0.027 of
            # the paper's D2Q5 runs diverges within 500 steps, s2 >= 1.2 is
            # stable through 5000 (probe at the same cell Reynolds number)
            spec.s2 = 1.5
        ref = {}
        for st in ("f64", "f32", "f16dev", "bf16dev"):
            dt = torch.float64 if st == "f64" else torch.float32
            solver = mdf.Solver([spec], storage=st, device=dev, stream=stream, u_ref=0.05,
                                init=("fields", [init64.to(dt)]))
            rec = {"Re": Re, "N": N, "s1": spec.s1, "s2": spec.s2 if spec.s2 > 0 else 8 * (2 - spec.s1) / (8 - spec.s1),
                   "storage": st, "errors": {}}
            t_total, done = 0.0, 0
            for t in steps:
                e0 = torch.cuda.Event(enable_timing=True)
                e1 = torch.cuda.Event(enable_timing=True)
                e0.record(stream)
                solver.step(t - done)
                e1.record(stream)
                torch.cuda.synchronize()
                t_total += e0.elapsed_time(e1) / 1e3
                done = t
                f = solver.fields(fields)
                torch.cuda.synchronize()
                cur = {"u": f["u"].double(), "P": f["P"].double(), "vort": f["vort"].double()}
                finite = all(bool(torch.isfinite(v).all()) for v in cur.values())
                if st == "f64":
                    ref[t] = cur
                    rec["errors"][str(t)] = {"finite": finite,
                                             "u_rms": float(cur["u"].pow(2).mean().sqrt())}
                else:
                    uscale = torch.linalg.vector_norm(ref[t]["u"].reshape(-1)).item()
                    rec["errors"][str(t)] = {
                        "finite": finite,
                        "u": _rel(ref[t]["u"], cur["u"]),
                        "P": _rel(ref[t]["P"], cur["P"], scale=uscale),
                        "vort": _rel(ref[t]["vort"], cur["vort"]),
                    }
            rec["ms_per_step"] = round(t_total * 1e3 / steps[-1], 4)
            rec["MLUPS"] = round(spec.nodes * steps[-1] / t_total / 1e6, 1)
            res.append(rec)
            print(json.dumps(rec), flush=True)
            del solver
            torch.cuda.empty_cache()
        ref.clear()
    with open(out_path, "w") as fh:
        json.dump(res, fh, indent=1)


def batch_study(out_path, ncases=512, max_steps=400000, wall_budget_s=420.0):
    """The seeded uneven batch: 512 cavity/channel cases, N in {64..512},
    Re log-uniform in [10, 1000], FP32, batched launches; autotuned launch
    shape, throughput, then every case run to residual
    1e-8 (checked every 100 steps)."""
    import numpy as np
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    bc = C.batch_cases(n=ncases)
    specs = [c.spec for c in bc]
    nodes = sum(s.nodes for s in specs)
    t0 = time.perf_counter()
    solver = mdf.Solver(specs, storage="f32", device=dev, stream=stream)
    chosen, tuned_ms = solver.autotune(trial_steps=20)
    torch.cuda.synchronize()
    rec = {"cases": ncases, "nodes": nodes, "autotune_shape": chosen, "autotune_ms_per_step": tuned_ms}
    n = 500
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    solver.step(n)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / n
    rec["throughput_MLUPS"] = round(nodes / ms / 1e3, 1)
    rec["ms_per_batched_step"] = round(ms, 4)
    print(json.dumps(rec), flush=True)
    t1 = time.perf_counter()
    # windows of run_steady: finished cases are retired between windows and
    # progress is reported (the residual snapshot carries over)
    n = len(specs)
    st = np.full(n, 2)
    steps = np.zeros(n, np.int64)
    res = np.full(n, np.inf)
    active = np.ones(n, bool)
    window, done = 20000, 0
    while active.any() and done < max_steps and time.perf_counter() - t1 < wall_budget_s:
        solver.set_active(active)
        w_st, w_steps, w_res = solver.run_steady(1e-8, 100, min(window, max_steps - done))
        done += window
        for k in np.nonzero(active)[0]:
            steps[k] += w_steps[k]
            res[k] = w_res[k]
            if w_st[k] in (0, 1):
                st[k] = w_st[k]
                active[k] = False
        print(json.dumps({"progress_steps": done, "converged": int((st == 0).sum()),
                          "nonfinite": int((st == 1).sum()), "running": int(active.sum()),
                          "running_nodes": int(sum(specs[k].nodes for k in np.nonzero(active)[0])),
                          "wall_s": round(time.perf_counter() - t1, 1)}), flush=True)
    wall = time.perf_counter() - t1
    node_steps = float(sum(sp.nodes * int(k) for sp, k in zip(specs, steps)))
    rec.update({
        "max_steps": max_steps, "wall_budget_s": wall_budget_s,
        "steady_wall_s": round(wall, 2),
        "init_to_steady_wall_s": round(time.perf_counter() - t0, 2),
        "converged": int((st == 0).sum()), "nonfinite": int((st == 1).sum()), "not_converged": int((st == 2).sum()),
        "steps_min": int(steps.min()), "steps_median": int(np.median(steps)), "steps_max": int(steps.max()),
        "node_steps": node_steps, "effective_MLUPS": round(node_steps / wall / 1e6, 1),
        "nonfinite_cases": [{"kind": bc[k].kind, "N": bc[k].N, "Re": round(bc[k].Re, 1), "U": round(bc[k].U, 4)}
                            for k in range(ncases) if st[k] == 1][:20],
        "unconverged_cases": [{"kind": bc[k].kind, "N": bc[k].N, "Re": round(bc[k].Re, 1),
                               "residual": float(res[k])} for k in range(ncases) if st[k] == 2][:20],
    })
    print(json.dumps(rec), flush=True)
    with open(out_path, "w") as fh:
        json.dump(rec, fh, indent=1)


def steady_study(out_path):
    """Wall time from initialisation to residual 1e-8 (K = 100) for the
    channel and the cavities of the benchmark configuration (FP32, vorticity
    and strain rate emitted by every launch for the cavities)."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    out = []
    runs = [("poiseuille 256x64", C.poiseuille_case(256, 64), 0),
            ("cavity 1024^2 Re=100", C.cavity_case(N=1024, Re=100.0), mdf.FIELD_VORT | mdf.FIELD_STRAIN),
            ("cavity 1024^2 Re=1000", C.cavity_case(N=1024, Re=1000.0), mdf.FIELD_VORT | mdf.FIELD_STRAIN)]
    for name, spec, fields in runs:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        solver = mdf.Solver([spec], storage="f32", device=dev, stream=stream)
        bufs = solver.new_field_buffers(fields) if fields else None
        st, steps, res = solver.run_steady(1e-8, 100, 5_000_000, fields, bufs)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        rec = {"case": name, "status": int(st[0]), "steps": int(steps[0]), "residual": float(res[0]),
               "wall_s": round(wall, 3), "MLUPS": round(spec.nodes * int(steps[0]) / wall / 1e6, 1)}
        print(json.dumps(rec), flush=True)
        out.append(rec)
    with open(out_path, "w") as fh:
        json.dump(out, fh, indent=1)


def warmstart_study(out_path, n_train=1024, n_test=32, N=128, epochs=30, batch=16, lr=2e-3, clip=None):
    """Learned warm start (cavities with obstacles, N^2): training data from
    the batched FP32 solver (residual 1e-7), training of the encoder-decoder
    with the project's kernels, then cold vs warm FP64 solves of held-out
    cases to residual 1e-8, and the ablation with f^eq-only warm starts."""
    import numpy as np
    import torch
    from paper_2108_08591_amd import nn
    from paper_2108_08591_amd import warmstart as WS
    log = lambda m: print(m, flush=True)
    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()
    rec = {"N": N, "n_train": n_train, "n_test": n_test, "epochs": epochs, "batch": batch}
    tr = WS.warmstart_cases(n_train, N, seed=20210819)
    te = WS.warmstart_cases(n_test, N, seed=20210820)
    solver, st, steps, res, wall = WS.solve(tr, "f32", tol=1e-7, max_steps=300000, stream=stream, log=log)
    good = [k for k in range(n_train) if st[k] == 0]
    rec.update({"datagen_wall_s": round(wall, 1), "datagen_converged": len(good),
                "datagen_nonfinite": int((st == 1).sum()), "datagen_steps_median": int(np.median(steps))})
    log(json.dumps({k: rec[k] for k in ("datagen_wall_s", "datagen_converged", "datagen_nonfinite")}))
    data = WS.dataset([tr[k] for k in good], _Subset(solver, good), log=log)
    del solver
    torch.cuda.empty_cache()
    # the last 64 converged cases are held out of training for the validation loss
    nv = min(64, len(good) // 8)
    val = {k: v[-nv:] for k, v in data.items()}
    data = {k: v[:-nv] for k, v in data.items()}
    model = nn.UNet(device="cuda:0", seed=0)
    rec["params"] = model.nparams
    rec.update({"lr": lr, "target_clip_sigma": clip, "n_val": nv})
    t0 = time.perf_counter()
    hist, vhist = WS.train(model, data, epochs=epochs, batch=batch, lr=lr, clip=clip, val=val, log=log)
    torch.cuda.synchronize()
    rec["train_wall_s"] = round(time.perf_counter() - t0, 1)
    rec["loss_history"] = [round(h, 6) for h in hist]
    rec["val_loss_history"] = vhist
    np.savez(os.path.join(os.path.dirname(out_path), f"warmstart_model_{N}.npz"), **model.state_dict())
    # held-out: cold vs warm, FP64
    cold, cst, csteps, cres, cwall = WS.solve(te, "f64", tol=1e-8, max_steps=600000, stream=stream, log=log)
    t0 = time.perf_counter()
    init = WS.predict(model, te, with_grad=True)
    torch.cuda.synchronize()
    t_inf = time.perf_counter() - t0
    # warm solves with the cold start from rest as the fallback (its steps and
    # wall time are charged to the warm side)
    where, wst, wsteps, wres, wwall, fallback = WS.solve_warm(te, init, "f64", tol=1e-8, max_steps=600000,
                                                              stream=stream, log=log)
    # an exact predictor: restart from the cold solution's own fields
    exact = [WS.solution_init(cold, k) for k in range(n_test)]
    _, xst, xsteps, _, xwall = WS.solve(te, "f64", tol=1e-8, max_steps=600000, init=exact, stream=stream, log=log)
    perr = [WS.prediction_error(init[k], exact[k], te[k]["mask"]) for k in range(n_test) if cst[k] == 0]
    init_eq = WS.predict(model, te, with_grad=False)
    weq, est, esteps, eres, ewall = WS.solve(te, "f64", tol=1e-8, max_steps=600000, init=init_eq, stream=stream,
                                             log=log)
    ok = [k for k in range(n_test) if cst[k] == 0 and wst[k] == 0]
    errs = [WS.field_error(cold, where[k][0], k, where[k][1]) for k in ok]
    cases_out = []
    for k in range(n_test):
        cases_out.append({"Re": round(te[k]["Re"], 1), "U": round(te[k]["U"], 4),
                          "obstacle_frac": round(float(te[k]["mask"].mean()), 4),
                          "cold_steps": int(csteps[k]), "warm_steps": int(wsteps[k]), "warm_feq_steps": int(esteps[k]),
                          "exact_restart_steps": int(xsteps[k]),
                          "cold_status": int(cst[k]), "warm_status": int(wst[k])})
    rec.update({
        "cold_wall_s": round(cwall, 2), "warm_wall_s": round(wwall + t_inf, 2), "inference_s": round(t_inf, 3),
        "warm_feq_wall_s": round(ewall + t_inf, 2),
        "speedup_wall": round(cwall / (wwall + t_inf), 3),
        "speedup_wall_note": "warm wall time includes inference and the cold re-solves of the fallback cases",
        "speedup_wall_target": 3.0,
        "fallback_cases": [int(k) for k in fallback],
        "speedup_steps_total": round(float(csteps[ok].sum()) / max(1.0, float(wsteps[ok].sum())), 3),
        "speedup_steps_median_case": round(float(np.median(csteps[ok] / np.maximum(wsteps[ok], 1))), 3),
        "ablation_feq_only_speedup_steps_total": round(float(csteps[ok].sum()) / max(1.0, float(esteps[ok].sum())), 3),
        "exact_fields_restart_speedup_steps_total": round(float(csteps[ok].sum()) / max(1.0, float(xsteps[ok].sum())), 3),
        "prediction_rel_l2_median": {c: float(np.median([e[c] for e in perr])) for c in WS.CHANNELS},
        "field_rel_l2_warm_vs_cold_max": max(errs) if errs else None,
        "field_rel_l2_warm_vs_cold_median": float(np.median(errs)) if errs else None,
        "fallbacks_needed": len(fallback),
        "warm_within_1e-4_of_cold": int(sum(1 for e in errs if e <= 1e-4)),
        "cases": cases_out,
    })
    log(json.dumps({k: v for k, v in rec.items() if k not in ("cases", "loss_history")}))
    with open(out_path, "w") as fh:
        json.dump(rec, fh, indent=1)


def _coarse_levels(cases, levels, stream, log=None):
    """The coarse solves of the coarse-informed warm start (FP32, residual
    1e-6): with levels = 1 the grid twice as coarse from rest; with levels =
    2 first the grid four times as coarse from rest, then the grid twice as
    coarse started from it.  Returns the twice-coarse cases, their solver and
    status and steps, the solutions interpolated to the fine grids (twice
    coarse, and four times coarse or None), the four-times-coarse steps (or
    None) and the wall time."""
    import numpy as np
    from paper_2108_08591_amd import warmstart as WS
    t0 = time.perf_counter()
    c2 = WS.coarse_cases(cases)
    up4 = None
    init2 = None
    steps4 = None
    if levels == 2:
        c4 = WS.coarse_cases(cases, factor=4)
        s4, st4, steps4, _, _ = WS.solve(c4, "f32", tol=1e-6, max_steps=300000, stream=stream, log=log)
        init2 = [u if u is not None else np.zeros((7, c["N"], c["N"]), np.float32)
                 for u, c in zip(WS.upsampled_init(c2, c4, s4, st4), c2)]
        up4 = WS.upsampled_init(cases, c4, s4, st4, factor=4)
        del s4
    s2, st2, steps2, _, _ = WS.solve(c2, "f32", tol=1e-6, max_steps=300000, init=init2, stream=stream, log=log)
    up2 = WS.upsampled_init(cases, c2, s2, st2)
    import torch
    torch.cuda.synchronize()
    return c2, s2, st2, steps2, up2, up4, steps4, time.perf_counter() - t0


def coarse_warmstart_study(out_path, n_train=4096, n_test=32, N=128, epochs=36, batch=16, lr=1e-3, levels=1):
    """Warm start informed by a coarse solve (an extension of the learned
    warm start): each case is first solved on a grid twice as coarse (FP32,
    residual 1e-6), its steady fields are interpolated to the fine grid, and
    the encoder-decoder, given them as extra inputs, predicts the correction
    to them.  With levels = 2 a grid four times as coarse is solved first; it
    starts the twice-coarse solve and is a second input of the network.
    Compared on held-out cases (FP64, residual 1e-8): cold start, the
    interpolated coarse solution alone (nested iteration, the method without
    the network), and coarse solution + network.  Warm wall times include
    the coarse solves and the inference."""
    import numpy as np
    import torch
    from paper_2108_08591_amd import nn
    from paper_2108_08591_amd import warmstart as WS
    log = lambda m: print(m, flush=True)
    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()
    rec = {"N": N, "n_train": n_train, "n_test": n_test, "epochs": epochs, "batch": batch, "lr": lr,
           "coarse_factor": 2, "coarse_levels": levels, "coarse_solve": "FP32, residual 1e-6"}
    tr = WS.warmstart_cases(n_train, N, seed=20210819)
    te = WS.warmstart_cases(n_test, N, seed=20210820)
    solver, st, steps, _, wall = WS.solve(tr, "f32", tol=1e-7, max_steps=300000, stream=stream, log=log)
    trc, csolver, cst, _, up_tr, up4_tr, _, cwall_tr = _coarse_levels(tr, levels, stream, log)
    del csolver
    good = [k for k in range(n_train) if st[k] == 0 and cst[k] == 0]
    rec.update({"datagen_wall_s": round(wall, 1), "coarse_datagen_wall_s": round(cwall_tr, 1),
                "train_cases_used": len(good)})
    log(json.dumps({k: rec[k] for k in ("datagen_wall_s", "coarse_datagen_wall_s", "train_cases_used")}))
    data = WS.dataset([tr[k] for k in good], _Subset(solver, good), log=log, coarse=[up_tr[k] for k in good],
                      coarse2=None if up4_tr is None else [up4_tr[k] for k in good])
    del solver, up_tr, up4_tr
    torch.cuda.empty_cache()
    nv = min(64, len(good) // 8)
    val = {k: v[-nv:] for k, v in data.items()}
    data = {k: v[:-nv] for k, v in data.items()}
    model = nn.UNet(device="cuda:0", seed=0)
    t0 = time.perf_counter()
    hist, vhist = WS.train(model, data, epochs=epochs, batch=batch, lr=lr, val=val, log=log)
    torch.cuda.synchronize()
    rec.update({"train_wall_s": round(time.perf_counter() - t0, 1), "loss_history": [round(h, 6) for h in hist],
                "val_loss_history": vhist})
    del data, val
    # held-out cases
    cold, cst_te, csteps, _, cwall = WS.solve(te, "f64", tol=1e-8, max_steps=600000, stream=stream, log=log)
    tec, cs_te, cst2, csteps2, up_te, up4_te, csteps4, t_coarse = _coarse_levels(te, levels, stream)
    t0 = time.perf_counter()
    pred = WS.predict(model, te, with_grad=True, coarse=up_te, coarse2=up4_te)
    torch.cuda.synchronize()
    t_inf = time.perf_counter() - t0
    rest = np.zeros((7, N, N))
    # a case whose coarse solve failed starts from rest
    init_nested = [u if u is not None else rest for u in up_te]
    init_net = [pred[k] if up_te[k] is not None else rest for k in range(n_test)]
    nst_s, nst, nsteps, _, nwall = WS.solve(te, "f64", tol=1e-8, max_steps=600000, init=init_nested, stream=stream)
    where, wst, wsteps, _, wwall, fallback = WS.solve_warm(te, init_net, "f64", tol=1e-8, max_steps=600000,
                                                           stream=stream)
    exact = [WS.solution_init(cold, k) for k in range(n_test)]
    ok = [k for k in range(n_test) if cst_te[k] == 0 and wst[k] == 0 and nst[k] == 0]
    coarse_equiv = float(csteps2.sum()) / 4.0          # coarse node-steps in fine node-steps
    if csteps4 is not None:
        coarse_equiv += float(csteps4.sum()) / 16.0
    perr_net = [WS.prediction_error(init_net[k], exact[k], te[k]["mask"]) for k in ok]
    perr_nest = [WS.prediction_error(init_nested[k], exact[k], te[k]["mask"]) for k in ok]
    errs = [WS.field_error(cold, where[k][0], k, where[k][1]) for k in ok]
    cs_ok = float(csteps[ok].sum())
    rec["cases"] = [{"Re": round(te[k]["Re"], 1), "Re_coarse": round(tec[k]["Re"], 1), "U": round(te[k]["U"], 4),
                     "cold_steps": int(csteps[k]), "coarse_steps": int(csteps2[k]), "coarse_status": int(cst2[k]),
                     "nested_steps": int(nsteps[k]), "network_steps": int(wsteps[k]),
                     "cold_status": int(cst_te[k]), "network_status": int(wst[k])} for k in range(n_test)]
    rec["speedup_fine_steps_network_median_case"] = round(float(np.median(csteps[ok] / np.maximum(wsteps[ok], 1))), 3)
    rec["speedup_fine_steps_nested_median_case"] = round(float(np.median(csteps[ok] / np.maximum(nsteps[ok], 1))), 3)
    rec.update({
        "cold_wall_s": round(cwall, 2), "coarse_wall_s": round(t_coarse, 2), "inference_s": round(t_inf, 3),
        "nested_fine_wall_s": round(nwall, 2), "network_fine_wall_s": round(wwall, 2),
        "speedup_wall_nested": round(cwall / (t_coarse + nwall), 3),
        "speedup_wall_network": round(cwall / (t_coarse + t_inf + wwall), 3),
        "network_fallback_cases": [int(k) for k in fallback],
        "speedup_fine_steps_nested": round(cs_ok / max(1.0, float(nsteps[ok].sum())), 3),
        "speedup_fine_steps_network": round(cs_ok / max(1.0, float(wsteps[ok].sum())), 3),
        "speedup_steps_incl_coarse_network": round(float(csteps.sum()) / (float(wsteps.sum()) + coarse_equiv), 3),
        "prediction_rel_l2_median_nested": {c: float(np.median([e[c] for e in perr_nest])) for c in WS.CHANNELS},
        "prediction_rel_l2_median_network": {c: float(np.median([e[c] for e in perr_net])) for c in WS.CHANNELS},
        "coarse_failed": int(sum(1 for u in up_te if u is None)),
        "warm_not_converged": int(sum(1 for k in range(n_test) if wst[k] != 0)),
        "field_rel_l2_warm_vs_cold_max": max(errs) if errs else None,
        "warm_within_1e-4_of_cold": int(sum(1 for e in errs if e <= 1e-4)), "compared_cases": len(ok),
    })
    log(json.dumps({k: v for k, v in rec.items() if k not in ("loss_history", "cases")}))
    with open(out_path, "w") as fh:
        json.dump(rec, fh, indent=1)


def restart_study(out_path, n=16, N=128):
    """What a warm start gains as a function of the accuracy of the fields it
    starts from: held-out cavities are solved cold to residual 1e-8 (FP64),
    refined to 1e-12, and restarted from the refined (P, u, grad u) exactly,
    with f^eq only, with P zeroed, and with seeded smooth relative errors of
    1e-4 .. 1e-1 on every channel or on the velocity alone."""
    import numpy as np
    import torch
    from paper_2108_08591_amd import warmstart as WS
    log = lambda m: print(m, flush=True)
    stream = torch.cuda.Stream()
    cases = [c for c in WS.warmstart_cases(24, N, seed=777) if c["Re"] < 600][:n]
    cold_solver, st, cold, _, wall = WS.solve(cases, "f64", 1e-8, 100, 400000, stream=stream)
    rec = {"N": N, "cases": len(cases), "cold_steps": cold.tolist(), "cold_status": st.tolist(),
           "cold_wall_s": round(wall, 2), "variants": []}
    first = [WS.solution_init(cold_solver, k) for k in range(len(cases))]
    del cold_solver
    ref_solver, st2, _, _, _ = WS.solve(cases, "f64", 1e-12, 100, 800000, init=first, stream=stream)
    ref = [WS.solution_init(ref_solver, k) for k in range(len(cases))]
    del ref_solver
    rng = np.random.default_rng(1)

    def smooth(n_):
        k = np.fft.fftfreq(n_)[:, None] ** 2 + np.fft.fftfreq(n_)[None, :] ** 2
        z = np.fft.ifft2(np.fft.fft2(rng.standard_normal((n_, n_))) * np.exp(-k * (n_ / 8) ** 2)).real
        return z / np.abs(z).max()

    def run(name, make, feq_only=False):
        init = []
        for k, c in enumerate(cases):
            a = make(ref[k].copy())
            a[:, c["mask"].astype(bool)] = 0.0
            init.append(a[:3].copy() if feq_only else a)
        _, wst, steps, _, w = WS.solve(cases, "f64", 1e-8, 100, 400000, init=init, stream=stream)
        ent = {"variant": name, "steps": steps.tolist(), "status": wst.tolist(),
               "speedup_steps_total": round(float(cold.sum()) / max(1.0, float(steps.sum())), 3)}
        rec["variants"].append(ent)
        log(json.dumps({k: ent[k] for k in ("variant", "speedup_steps_total")}))

    run("exact", lambda a: a)
    run("exact, f^eq only", lambda a: a, feq_only=True)
    run("exact, P = 0", lambda a: np.concatenate([0 * a[:1], a[1:]]))
    for eps in (1e-4, 1e-3, 1e-2, 1e-1):
        def all_ch(a, eps=eps):
            for ch in range(a.shape[0]):
                a[ch] *= 1 + eps * smooth(N)
            return a

        def vel(a, eps=eps):
            scale = np.abs(a[1:3]).max()
            a[1] += eps * scale * smooth(N)
            a[2] += eps * scale * smooth(N)
            return a
        run(f"every channel x (1 + {eps:g} s)", all_ch)
        run(f"u, v + {eps:g} max|u| s", vel)
    with open(out_path, "w") as fh:
        json.dump(rec, fh, indent=1)


class _Subset:
    """Read-outs of selected cases of a solver, renumbered from 0."""

    def __init__(self, solver, idx):
        self.solver, self.idx = solver, idx

    def fields(self, fields, k):
        return self.solver.fields(fields, self.idx[k])


def _launch_ms(solver, stream, nsteps, reps=5):
    """HIP-event time of one call of nsteps steps on the solver's stream
    (no other work in between), median of reps, in ms."""
    import statistics
    import torch
    res = []
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        solver.step(nsteps)
        e1.record(stream)
        torch.cuda.synchronize()
        res.append(e0.elapsed_time(e1))
    return statistics.median(res)


def several_steps(storage, state_bytes):
    """Steps per launch and kernel of the 2D form with several steps per
    launch, for a context whose two population buffers hold `state_bytes`:
    tiles of four steps in FP64 and inside the 256 MB Infinity Cache, strips
    of five (FP32) or four steps beyond it."""
    strips = storage != "f64" and state_bytes > 256 << 20
    return (5 if strips and storage == "f32" else 4), ("k_march" if strips else "k_tile")


def launch_bytes(nodes, state_bytes, field_bytes, steps):
    """Bytes of one launch of `steps` steps: (algorithmic, physical).  The state
    counts once per step and, physically, once per launch; emitted fields are
    written once per launch, at its last step."""
    return nodes * (state_bytes * steps + field_bytes), nodes * (state_bytes + field_bytes)


def batch_headline(args, dev, stream):
    """The headline: the seeded 512-case uneven batch (2D cavities and
    channels, N in {64, 96, ..., 512}, 53.6 M nodes, the largest
    configuration that fits one GPU) in the paper's FP64, in batched launches
    of one step or, where the autotuner picks it, of several, with
    the FP64 K-interval residual fused into the last step of every 100."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf

    bcs = C.batch_cases(n=512)
    specs = [b.spec for b in bcs]
    nodes = sum(sp.nodes for sp in specs)
    solver = mdf.Solver(specs, storage=args.storage, device=dev, stream=stream, sets=args.sets)
    nsets = solver.nsets
    sbytes = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}[args.storage]
    chosen, tuned_ms = solver.autotune(trial_steps=10)
    bx, by, groups, form = chosen
    K = 100
    solver.run_steady(1e-300, K, max(args.warmup, 1))     # warm-up and the first residual snapshot
    torch.cuda.synchronize()

    # timed region: whole job, inputs resident in HBM
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev0.record(stream)
    status, steps_done, res = solver.run_steady(1e-300, K, args.steps)
    ev1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    gpu_ms = ev0.elapsed_time(ev1)
    assert all(int(k) == args.steps for k in steps_done), steps_done
    nonfinite = int((status == 1).sum())
    elapsed = max(wall, gpu_ms / 1e3)
    mlups = nodes * args.steps / elapsed / 1e6

    # average launch duration of the dominant kernel, HIP events on its
    # stream: a call of 201 steps is 200 / s launches of s steps and one
    # one-step launch (a chunk graph), a call of 1 step one one-step launch
    step_bytes = 2 * 5 * nsets * sbytes            # one read and one write of the state per node and step
    if form == 2:
        steps_per_launch, kname = several_steps(args.storage, nodes * step_bytes)
        m = 200 // steps_per_launch
        t_long = _launch_ms(solver, stream, 201)
        t_one = _launch_ms(solver, stream, 1)
        avg_ms = (t_long - t_one) / m
        kernel = f"{kname}_batch<D2Q5{'' if nsets == 3 else 'V'},{args.storage.upper()}>"
        timing = f"HIP events, (time of 201 steps - time of 1 step) / {m}, median of 5"
    else:
        avg_ms = _launch_ms(solver, stream, 200) / 200
        steps_per_launch = 1
        kernel = f"k_step_batch<D2Q5{'' if nsets == 3 else 'V'},{args.storage.upper()}>"
        timing = "HIP events around 200 back-to-back steps, median of 5"
    # per-step bytes x node-steps of one launch; one read and one write of the state per launch
    alg_bytes, phys_bytes = launch_bytes(nodes, step_bytes, 0, steps_per_launch)
    achieved = alg_bytes / (avg_ms / 1e3) / 1e9
    phys = phys_bytes / (avg_ms / 1e3) / 1e9
    kernel_key = f"{kernel}_c4_512"
    traffic = measured_traffic(kernel_key, alg_bytes)
    return {
        "metric": "MLUPS (lattice-node updates per second, millions)",
        "value": round(mlups, 1),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(elapsed * 1e3 / args.steps, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if args.storage == "f64" else "f32",
        "data": "synthetic",
        "config": {
            "workload": f"512 seeded uneven 2D cases (cavity/channel, N in 64..512 step 32, Re log-uniform "
                        f"10..1000, U 0.05..0.1), {nodes / 1e6:.1f} M nodes, D2Q5 x {nsets} sets, "
                        f"{args.storage.upper()} storage, batched launches, FP64 "
                        f"residual every {K} steps",
            "cases": len(specs), "nodes": nodes, "storage": args.storage, "sets": args.sets,
            "launch": f"{bx}x{by}g{groups}{'svt'[form]} (autotuned)",
            "nonfinite_cases": nonfinite,
        },
        # measured bytes over time of the dominant kernel on a working set of
        # 2 x state (beyond the 256 MB Infinity Cache), against the HBM peak
        "hbm_roofline_pct": round(100.0 * phys / HBM_PEAK_GBS, 2),
        # the same launches counted in one-step bytes per node-step
        "one_step_equiv_pct": round(100.0 * mlups * 1e6 * step_bytes / (HBM_PEAK_GBS * 1e9), 2),
        "roofline": {
            "bound": "hbm",
            "achieved": round(achieved, 1),
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": round(achieved / HBM_PEAK_GBS, 4),
            "traffic": traffic,
            "kernel": kernel,
            "bytes_per_launch": alg_bytes,
            "steps_per_launch": steps_per_launch,
            "avg_launch_ms": round(avg_ms, 5),
            "launch_timing": timing,
            "hbm_physical": {"bytes_per_launch": phys_bytes, "achieved": round(phys, 1),
                             "frac": round(phys / HBM_PEAK_GBS, 4)},
            "note": ("achieved counts the per-step algorithmic bytes (one read and one write of the state per "
                     "node-step) of every node-step a launch performs; with several steps per launch the state "
                     "crosses HBM once per launch, so frac may exceed 1; hbm_physical counts one read and "
                     f"one write of the state per launch; working set {2 * phys_bytes / 2 ** 30:.1f} GiB"),
        },
        "residual_median": float(sorted(res)[len(res) // 2]),
    }


def cavity_leg(args, dev, stream, N, nsteps):
    """The lid-driven cavity of the channel-and-cavity configuration, FP32,
    Re = 1000, lid 0.1, vorticity and strain rate emitted by every launch, in
    the given launch shape: MLUPS and the step kernel's roofline."""
    import torch
    from paper_2108_08591_amd import cases as C
    from paper_2108_08591_amd import mdf

    spec = C.cavity_case(N=N, Re=1000.0, U=0.1)
    fields = mdf.FIELD_VORT | mdf.FIELD_STRAIN
    solver = mdf.Solver([spec], storage="f32", device=dev, stream=stream, sets=args.sets)
    nsets = solver.nsets
    bx, by, groups, form = parse_launch(args.launch)
    solver.set_launch(bx, by, groups, form)
    out = solver.new_field_buffers(fields)
    solver.run_steady(1e-300, 100, 200, fields, out)
    torch.cuda.synchronize()
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    status, steps_done, res = solver.run_steady(1e-300, 100, nsteps, fields, out)
    ev1.record(stream)
    torch.cuda.synchronize()
    mlups = spec.nodes * nsteps / (ev0.elapsed_time(ev1) / 1e3) / 1e6
    state_bytes = 2 * 5 * nsets * 4
    field_bytes = 4 * 4
    steps_per_launch, kname = several_steps("f32", spec.nodes * state_bytes) if form == 2 else (1, "k_step")
    # a call of 20 m + 1 steps ends with a launch of one step
    nt = (201 if N <= 2048 else 41) if form == 2 else 200
    if form == 2:
        t_long, t_one = (time_launches(solver, stream, n, fields, out, 5) * n for n in (nt, 1))
        avg_ms = (t_long - t_one) * steps_per_launch / (nt - 1)
    else:
        avg_ms = time_launches(solver, stream, nt, fields, out, 5)
    alg_bytes, phys_bytes = launch_bytes(spec.nodes, state_bytes, field_bytes, steps_per_launch)
    rec = {"MLUPS": round(mlups, 1), "nodes": spec.nodes, "steps": nsteps,
           "launch": f"{bx}x{by}g{groups}{'svt'[form]}",
           "kernel": f"{kname}<D2Q5{'' if nsets == 3 else 'V'},F32,emit>",
           "avg_launch_ms": round(avg_ms, 5), "bytes_per_launch": alg_bytes,
           "roofline_frac": round(alg_bytes / (avg_ms / 1e3) / 1e9 / HBM_PEAK_GBS, 4),
           "steps_per_launch": steps_per_launch,
           "hbm_physical_frac": round(phys_bytes / (avg_ms / 1e3) / 1e9 / HBM_PEAK_GBS, 4),
           "working_set_MiB": (state_bytes * spec.nodes) >> 20}
    del solver, out
    torch.cuda.empty_cache()
    return rec


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--headline-only", action="store_true",
                    help="time only the 512-case FP64 batch (no cavity legs, no device copy)")
    ap.add_argument("--storage", default="f64", choices=["f64", "f32", "f16dev", "bf16dev"],
                    help="storage of the batch leg (the configuration's arithmetic is FP64)")
    ap.add_argument("--sets", default="all", choices=["all", "velocity"],
                    help="distribution sets stored: all d+1 (the configuration) or the d velocity sets (Remark IV)")
    ap.add_argument("--launch", default="128x2g8t",
                    help="cavity legs: threads per block, XCD groups and kernel form, BXxBYgG[s|v|t] (s: one node/thread, v: vector, t: several steps per launch)")
    ap.add_argument("--variants-study", metavar="OUT_JSONL",
                    help="velocity sets / Scheme II / force field against the plain update")
    ap.add_argument("--sweep", metavar="OUT_JSONL",
                    help="time the step kernel over grid sizes, storages and launch shapes")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain copy of known size (traffic-counter calibration)")
    ap.add_argument("--summarize-trace", nargs=2, metavar=("DB", "OUT_MD"),
                    help="write a markdown summary of a rocprofv3 kernel-trace database")
    ap.add_argument("--summarize-traffic", nargs=5,
                    metavar=("FETCH_DB", "WRITE_DB", "COPY_FETCH_DB", "COPY_WRITE_DB", "OUT_MD"),
                    help="calibrated HBM traffic of the step kernel from rocprofv3 counter databases")
    ap.add_argument("--command", default="", help="command recorded in a summary")
    ap.add_argument("--traffic-kernel", default="batch2", choices=["batch2", "step2z", "step2"],
                    help="kernel whose counters --summarize-traffic reads: the headline's batched tile "
                         "kernel, the 3D two-step kernel, or the 1024^2 cavity's tile kernel")
    ap.add_argument("--tgv3d", nargs="+", metavar="STORAGE FORM [GROUPS [BX BY]]",
                    help="time the 3D Taylor-Green step kernel (256^3) in one storage and form (XCD groups, "
                         "default 8; block, default 64 x 4)")
    ap.add_argument("--grid2d", nargs="+", metavar="STORAGE FORM [N [GROUPS]]",
                    help="time the 2D cavity step kernel (D2Q5 x 3 sets, default 8192^2, no emission) in one "
                         "storage and form")
    ap.add_argument("--summarize-counters", nargs="+", metavar="DB",
                    help="markdown summary of rocprofv3 --pmc databases: OUT_MD KERNEL_PREFIX NODE_STEPS DB...")
    ap.add_argument("--conv-study", metavar="OUT_JSONL",
                    help="the warm-start network's 3x3 convolutions at 256^2, batch 16: TFLOP/s per layer")
    ap.add_argument("--lattice-per-set-study", metavar="OUT_JSONL",
                    help="a lattice per set against the plain D2Q9 / D3Q15 (one node per thread)")
    ap.add_argument("--precision-study", metavar="OUT_JSON", help="FP16/BF16/FP32 vs FP64 storage, 3D TGV")
    ap.add_argument("--batch-study", metavar="OUT_JSON", help="512-case uneven batch to steady state")
    ap.add_argument("--batch-max-steps", type=int, default=400000)
    ap.add_argument("--batch-wall-s", type=float, default=420.0)
    ap.add_argument("--steady-study", metavar="OUT_JSON", help="wall time to residual 1e-8")
    ap.add_argument("--warmstart-study", metavar="OUT_JSON", help="learned warm start vs cold start")
    ap.add_argument("--restart-study", metavar="OUT_JSON", help="warm-start gain vs accuracy of the initial fields")
    ap.add_argument("--coarse-warmstart-study", metavar="OUT_JSON",
                    help="warm start from a coarse solve, with and without the network's correction")
    ap.add_argument("--ws-train", type=int, default=1024)
    ap.add_argument("--ws-epochs", type=int, default=30)
    ap.add_argument("--ws-n", type=int, default=128)
    ap.add_argument("--ws-lr", type=float, default=1e-3)
    ap.add_argument("--ws-batch", type=int, default=16)
    ap.add_argument("--ws-clip", type=float, default=0.0, help="target clip in standard deviations (0: none)")
    ap.add_argument("--ws-levels", type=int, default=1, choices=[1, 2],
                    help="coarse-informed warm start: coarse grids solved first (2: four and two times coarser)")
    args = ap.parse_args()
    if args.copy_calibration:
        copy_calibration()
        return
    if args.variants_study:
        variants_study(args.variants_study)
        return
    if args.sweep:
        sweep(args.sweep)
        return
    if args.precision_study:
        precision_study(args.precision_study)
        return
    if args.batch_study:
        batch_study(args.batch_study, max_steps=args.batch_max_steps, wall_budget_s=args.batch_wall_s)
        return
    if args.steady_study:
        steady_study(args.steady_study)
        return
    if args.coarse_warmstart_study:
        coarse_warmstart_study(args.coarse_warmstart_study, n_train=args.ws_train, N=args.ws_n,
                               epochs=args.ws_epochs, lr=args.ws_lr, batch=args.ws_batch, levels=args.ws_levels)
        return
    if args.restart_study:
        restart_study(args.restart_study)
        return
    if args.warmstart_study:
        warmstart_study(args.warmstart_study, n_train=args.ws_train, N=args.ws_n, epochs=args.ws_epochs,
                        lr=args.ws_lr, clip=args.ws_clip or None, batch=args.ws_batch)
        return
    if args.conv_study:
        conv_study(args.conv_study)
        return
    if args.lattice_per_set_study:
        lattice_per_set_study(args.lattice_per_set_study)
        return
    if args.tgv3d:
        tgv3d_timing(args.tgv3d[0], int(args.tgv3d[1]), groups=int(args.tgv3d[2]) if len(args.tgv3d) > 2 else 8,
                     bx=int(args.tgv3d[3]) if len(args.tgv3d) > 4 else 64,
                     by=int(args.tgv3d[4]) if len(args.tgv3d) > 4 else 4)
        return
    if args.grid2d:
        g = args.grid2d
        grid2d_timing(g[0], int(g[1]), N=int(g[2]) if len(g) > 2 else 8192, groups=int(g[3]) if len(g) > 3 else 8)
        return
    if args.summarize_counters:
        out_md, prefix, node_steps = args.summarize_counters[:3]
        with open(out_md, "w") as fh:
            fh.write(summarize_counters(args.summarize_counters[3:], args.command, int(node_steps), prefix))
        return
    if args.summarize_trace:
        with open(args.summarize_trace[1], "w") as fh:
            fh.write(summarize_trace(args.summarize_trace[0], args.command))
        return
    if args.summarize_traffic:
        fdb, wdb, cfdb, cwdb, out_md = args.summarize_traffic
        if args.traffic_kernel == "batch2":
            # the headline's dominant kernel: four-step batched launches of the
            # 512-case FP64 batch (no emission, no masks, non-temporal stores,
            # 32-bit node offsets); per-step algorithmic bytes of both steps
            from paper_2108_08591_amd import cases as C
            nodes = sum(b.spec.nodes for b in C.batch_cases(n=512))
            md, ent = summarize_traffic(fdb, wdb, cfdb, cwdb, "k_tile_batch<LatD2Q5, 0, true, 4, false, false, false>",
                                        nodes * 4 * (2 * 15 * 8), "k_tile_batch<D2Q5,F64>_c4_512",
                                        args.command.split(" ;; "))
        elif args.traffic_kernel == "step2z":
            # the 3D Taylor-Green kernel at 256^3, two steps per launch, FP32
            nodes = 256 ** 3
            md, ent = summarize_traffic(fdb, wdb, cfdb, cwdb, "k_step2z<LatD3Q7, 1, false, false, true, false>",
                                        nodes * 2 * (2 * 28 * 4), "k_step2z<D3Q7,F32>_tgv256",
                                        args.command.split(" ;; "))
        else:
            nodes = 1024 * 1024
            md, ent = summarize_traffic(fdb, wdb, cfdb, cwdb, "k_tile<LatD2Q5, 1, true, 4, false, true, false>",
                                        nodes * (2 * 15 * 4 + 4 * 4), "k_tile<D2Q5,F32,emit>_cavity1024",
                                        args.command.split(" ;; "))
        with open(out_md, "w") as fh:
            fh.write(md)
        path = os.path.join(ROOT, "profiles", "traffic_counters.json")
        data = json.load(open(path)) if os.path.exists(path) else {}
        data.update(ent)
        with open(path, "w") as fh:
            json.dump(data, fh, indent=1)
        return
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU; the multi-GPU path is a design "
                                   "(slab decomposition with halo exchange) and is not built",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.Stream(device=dev)
    result = batch_headline(args, dev, stream)
    if not args.headline_only:
        result["cavity1024_f32"] = cavity_leg(args, dev, stream, 1024, 4000)
        result["cavity8192_f32"] = cavity_leg(args, dev, stream, 8192, 41)
        # the 3D Taylor-Green vortex of the precision configuration at 256^3 in
        # each storage, in the form and launch shape the autotuner picks
        result["tgv3d256"] = {st: tgv3d_timing(st, None, quiet=True, tune=True) for st in ("f64", "f32", "f16dev")}
        result["device_copy"] = device_copy_bandwidth()
    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline_batch()
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
