#!/usr/bin/env python3
"""Benchmark: full-state sweep of a random lattice circuit on one MI355X.

One step = the whole hot path over one synthetic circuit instance:
circuit_create (host) -> pass planning (host) -> sv_simulate: |+>^n (layer 0)
generated by the first fused pass, layers 1..d in all fused passes, FP64
norm accumulated by the last pass, gather of 4096 sampled amplitudes.  Default workload: 30 qubits on a
5x6 lattice, depth 20 (full 2^30 complex64 state, 8 GiB).

value = amplitude updates per second = G * 2^n / step time, G = gates of the
circuit including layer 0.  The JSON line also carries the roofline of the
dominant kernel (the fused tile pass: 16 bytes of algorithmic HBM traffic
per amplitude per pass, timed with HIP events on the launch stream), the
unfused comparator path on the same workload, the sampled amplitude error
against stored oracle values, and the CPU oracle timed on a bounded sample.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = ("amplitude-updates/s & HBM GB/s (% peak), batched vs plain, "
          "at ≤1e-5 amp error")
HBM_PEAK_GBPS = 8000.0


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=20)
    p.add_argument("--warmup", type=int, default=3)
    p.add_argument("--workload", default="6x6m2-d30",
                   help="sweep workload (6x6m2-d30, 5x6-d20, 4x5-d10) or a mode: precision, "
                        "7x7-d16, uneven, task2, combine, partition")
    p.add_argument("--secondary", default="5x6-d20",
                   help="sweep workload also timed and reported under 'secondary' ('' = none)")
    p.add_argument("--reg", type=int, default=0, help="register qubits (0 = default)")
    p.add_argument("--thr", type=int, default=0, help="thread qubits (0 = default)")
    p.add_argument("--low", type=int, default=0, help="low resident qubits (0 = default)")
    p.add_argument("--jit", type=int, default=0,
                   help="pass kernels: 1 one tile per workgroup, 2 persistent, -1 generic (0 = library)")
    p.add_argument("--pass-forms", type=int, default=0,
                   help="with --jit 3: bit p set = pass p runs persistent")
    p.add_argument("--no-plain", action="store_true", help="skip the unfused comparator")
    p.add_argument("--no-tune", action="store_true",
                   help="skip the autotuner (default shape unless --reg/--thr/--low)")
    p.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    p.add_argument("--cpu-seconds", type=float, default=12.0)
    p.add_argument("--traffic-json", default=os.path.join(ROOT, "profiles", "traffic.json"))
    p.add_argument("--count", type=int, default=512, help="circuits of the uneven batch")
    p.add_argument("--dense-k", type=int, default=6, help="precision form: dense block width")
    p.add_argument("--wave", type=int, default=32, help="7x7 split: 28-qubit branches per batch")
    p.add_argument("--a-waves", type=int, default=4,
                   help="7x7 split: timed batches of 28-qubit branches (bounded sample)")
    p.add_argument("--oracle-max-n", type=int, default=26,
                   help="uneven batch: check circuits up to this size against the oracle")
    p.add_argument("--r0", type=int, default=2, help="partition: initial cut after row r0 - 1")
    p.add_argument("--max-move", type=int, default=3, help="partition: largest line offset")
    p.add_argument("--cpu-probe", type=float, default=0.0, help=argparse.SUPPRESS)
    p.add_argument("--calibrate-copy", action="store_true",
                   help="run one 1 GiB device copy first (counter calibration)")
    return p.parse_args()


def golden(name):
    path = os.path.join(ROOT, "tests", "golden", f"{name}_amplitudes.txt")
    if not os.path.exists(path):
        return None, None
    import numpy as np
    xs, amps = [], []
    for line in open(path):
        if line.startswith("#"):
            continue
        x, re, im = line.split()
        xs.append(int(x))
        amps.append(complex(float(re), float(im)))
    return np.array(xs, np.uint64), np.array(amps)


def cpu_baseline(spec, seconds, max_qubits=32):
    """The CPU oracle as it stands (complex128, gate by gate, OpenMP) on a
    bounded sample of the same workload: the first gates of the circuit on
    the full-size state, until `seconds` of work have been done.  A state the
    host cannot hold (16 * 2^n bytes above 64 GiB) is sampled on its low
    `max_qubits` qubits: the first gates of the circuit that act on those
    qubits only, on a 2^max_qubits complex128 state.  The state is allocated
    and touched before the clock starts."""
    import numpy as np
    from oracle import circuit as OC
    from oracle import sim
    from paper_1804_04797_amd import workloads
    lat = OC.Lattice(spec["rows"], spec["cols"], workloads.present_grid(spec))
    gates = OC.random_circuit(lat, spec["depth"], spec["seed"])
    n = lat.n
    note = f"the full 2^{n} complex128 state"
    if n > max_qubits:
        gates = [g for g in gates if g[1] < max_qubits and g[2] < max_qubits]
        note = (f"a 2^{max_qubits} complex128 state (the gates on qubits 0..{max_qubits - 1}; the "
                f"full 2^{n} state, {16 << (n - 30)} GiB, exceeds the host memory limit)")
        n = max_qubits
    psi = sim.zero_state(n)
    psi[:] = 0
    psi[0] = 1
    done = 0
    t0 = time.perf_counter()
    while done < len(gates) and time.perf_counter() - t0 < seconds:
        sim.run(psi, n, gates[done:done + 1])
        done += 1
    dt = time.perf_counter() - t0
    del psi
    return {"value": done * float(1 << n) / dt, "unit": "amplitude-updates/s",
            "cores": sim.threads(), "kind": "oracle",
            "sample": f"first {done} of {len(gates)} gates of {spec['name']} on {note} ({dt:.1f} s)"}


def cpu_single_thread(name, seconds):
    """The same oracle sample with one OpenMP thread, in a child process
    (the thread count is fixed when the OpenMP runtime starts), on at most
    30 qubits."""
    import subprocess
    env = dict(os.environ, OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, os.path.abspath(__file__), "--workload", name,
                        "--cpu-probe", str(seconds)], env=env, capture_output=True, text=True,
                       timeout=seconds * 10 + 300)
    for line in r.stdout.splitlines():
        if line.startswith("{"):
            return json.loads(line)
    return None


def _time_graph(fn, reps):
    import torch
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / reps


def _caches():
    """The on-disk caches this process uses (the library reads these
    variables): tuned options and compiled code objects, reused across
    processes."""
    return {k: os.environ.get(k) or None for k in ("QSV_TUNE_CACHE", "QSV_JIT_CACHE")}


def _progress(msg):
    """One line on stderr as a long stage of a run ends."""
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def uneven_setup(count, dev, m=16, stage=None):
    """The uneven batch as the benchmark runs it: count circuits of 14..26
    qubits, depth 8..24 (seeded), their states, m sampled bitstrings each,
    the size-class autotune (one representative per qubit count of the
    HBM-streaming class, 2^21 amplitudes or more, tuned on the device and its
    tile shape handed to the other circuits of its class), and the batch.
    Returns a dict of everything (also used by the parity tests, which pass
    `stage` to run it in steps: "tune" stops after the class autotune,
    ("compile", k, K) builds and runs the k-th of K groups of the compiled
    class as a batch of their own (their kernels are then cached for the
    full batch), "run" builds and runs the full batch)."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    if isinstance(stage, dict):  # continue from an earlier step
        U = stage
    else:
        U = _uneven_items(count, dev, m)
        _uneven_tune(U, dev)
        if stage == "tune":
            return U
    _uneven_run(U)
    return U


def _uneven_items(count, dev, m):
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    items = []
    for n, d, sd in workloads.uneven_batch(count):
        rows, cols, pres = workloads.lattice_for_qubits(n)
        items.append((qsv.circuit_create(rows, cols, pres, d, sd), n, d, sd))
    states = [torch.empty(1 << n, dtype=torch.complex64, device=dev) for _, n, _, _ in items]
    xs = np.concatenate([workloads.bitstrings(n, m, 1000 + i) for i, (_, n, _, _) in enumerate(items)])
    bits = torch.from_numpy(xs.view(np.int64)).to(dev)
    table = torch.empty(len(items) * m, dtype=torch.complex64, device=dev)
    return dict(items=items, states=states, xs=xs, bits=bits, table=table, m=m)


def _uneven_tune(U, dev):
    import torch
    from paper_1804_04797_amd import qsv
    items = U["items"]
    t_tune = time.perf_counter()
    class_tiles = {}
    for c, n, _, _ in items:
        if n >= 21 and n not in class_tiles:
            scratch = torch.empty(1 << n, dtype=torch.complex64, device=dev)
            class_tiles[n], _ = qsv.sv_tune(scratch, c, layer_begin=1)
            del scratch
            _progress(f"class autotune: {n} qubits -> {class_tiles[n]}")
    for c, n, _, _ in items:
        if n in class_tiles:
            qsv.sv_tune_set(c, class_tiles[n], layer_begin=1)
    U["class_tiles"] = class_tiles
    U["tune_s"] = time.perf_counter() - t_tune


def uneven_precompile(U, k, K):
    """Build and run, as a batch of its own, the k-th of K groups of the
    compiled class (2^21 amplitudes or more): compiles their pass kernels,
    which the full batch then finds in the library's cache."""
    import torch
    from paper_1804_04797_amd import qsv
    big = [i for i, (_, n, _, _) in enumerate(U["items"]) if n >= 21]
    part = big[k::K]
    if not part:
        return 0
    b = qsv.sv_batch_create([U["items"][i][0] for i in part])
    qsv.sv_batch_run(b, [U["states"][i] for i in part], init_plus=True)
    torch.cuda.synchronize()
    return len(part)


def _uneven_run(U):
    import torch
    from paper_1804_04797_amd import qsv
    t0 = time.perf_counter()
    b = qsv.sv_batch_create([c for c, _, _, _ in U["items"]])
    qsv.sv_batch_run(b, U["states"], init_plus=True, bitstrings=U["bits"], m=U["m"], amp_table=U["table"])
    torch.cuda.synchronize()
    U["batch"] = b
    U["setup_s"] = time.perf_counter() - t0


def bench_uneven(a):
    """Uneven batch: independent circuits of 14..26 qubits, depth 8..24,
    swept by one graph launch (batched) against one sv_simulate call per
    circuit with the same per-circuit options (unbatched) and the per-gate
    path."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv
    dev = torch.device("cuda:0")
    U = uneven_setup(a.count, dev, stage="tune")
    t_setup = time.perf_counter()
    groups = 8
    for k in range(groups):  # compile the compiled class's kernels in groups
        uneven_precompile(U, k, groups)
        _progress(f"compiled group {k + 1} of {groups}")
    U = uneven_setup(a.count, dev, stage=U)
    U["setup_s"] = time.perf_counter() - t_setup
    _progress("batch built and run once")
    items, states, xs, bits, table, m, b = (U[k] for k in ("items", "states", "xs", "bits", "table", "m", "batch"))
    class_tiles, tune_s, setup_s = U["class_tiles"], U["tune_s"], U["setup_s"]
    au = sum(c.info()[2] * float(1 << n) for c, n, _, _ in items)
    tb = _time_graph(lambda: qsv.sv_batch_run(b, states, init_plus=True, bitstrings=bits, m=m,
                                              amp_table=table), a.steps)
    got = table.cpu().numpy()
    outs = [table[i * m:(i + 1) * m] for i in range(len(items))]
    _progress("batched runs timed")

    # the unbatched comparator runs every circuit with the options the batch
    # gives it: compiled kernels on the class-tuned tile from 2^21 amplitudes,
    # the generic kernel on the batch's tile below
    def per_circuit_opts(n):
        if n >= 21:
            t = class_tiles[n]
            return dict(reg_qubits=t["reg_qubits"], thread_qubits=t["thread_qubits"],
                        low_qubits=t["low_qubits"], plain=0, jit=1, out_of_place=-1)
        return dict(reg_qubits=5, thread_qubits=8, low_qubits=5, plain=0, jit=-1)
    copts = [per_circuit_opts(n) for _, n, _, _ in items]

    def unbatched():  # in place, no norm: no workspace
        for (c, n, _, _), st, o, i, co in zip(items, states, outs, range(len(items)), copts):
            qsv.sv_simulate(st, c, init_kind=qsv.INIT_PLUS, layer_begin=1, opts=co,
                            bitstrings=bits[i * m:(i + 1) * m], amps_out=o, workspace=False)
    unbatched()
    tu = _time_graph(unbatched, max(1, a.steps // 2))

    def unbatched_sweeps():  # the same calls without the gather (no bitstring range check, no wait)
        for (c, n, _, _), st, co in zip(items, states, copts):
            qsv.sv_simulate(st, c, init_kind=qsv.INIT_PLUS, layer_begin=1, opts=co, workspace=False)
    tus = _time_graph(unbatched_sweeps, max(1, a.steps // 2))
    plain_opts = {"reg_qubits": 0, "thread_qubits": 0, "low_qubits": 0, "plain": 1, "jit": 0}

    def plain():
        for (c, n, _, _), st in zip(items, states):
            qsv.sv_simulate(st, c, init_kind=qsv.INIT_PLUS, layer_begin=1, opts=plain_opts)
    tp = _time_graph(plain, 1)
    _progress("unbatched and per-gate comparators timed")
    # error distribution against the oracle (every circuit up to
    # --oracle-max-n qubits), per size class
    from oracle import circuit as OC
    from oracle import sim
    errs, per_class = [], {}
    for i, (c, n, d, sd) in enumerate(items):
        if n > a.oracle_max_n:
            continue
        psi = np.full(1 << n, 2.0 ** (-n / 2), np.complex128)
        g = [x for x in OC.random_circuit(OC.Lattice.for_qubits(n), d, sd) if x[3] >= 1]
        ref = sim.run(psi, n, g)[xs[i * m:(i + 1) * m]]
        e = float(np.max(np.abs(got[i * m:(i + 1) * m] - ref))) * 2 ** (n / 2)
        errs.append(e)
        k = "lds (n<=14)" if n <= 14 else ("generic (n<21)" if n < 21 else "compiled (n>=21)")
        pc = per_class.setdefault(k, {"checked": 0, "max_scaled": 0.0})
        pc["checked"] += 1
        pc["max_scaled"] = max(pc["max_scaled"], e)
        if len(errs) % 64 == 0:
            _progress(f"oracle checked {len(errs)} circuits")
    # algorithmic HBM bytes of one batched run: every pass of every circuit
    # reads and writes its state (16 B per amplitude), except the first,
    # which generates |+>^n and only writes (8 B)
    lds_shape = {14: (5, 9), 13: (5, 8), 12: (5, 7), 11: (4, 7)}

    def batch_opts(n):
        if n >= 21:
            return copts[[nn for _, nn, _, _ in items].index(n)]
        r, t = lds_shape.get(n, (5, 8))
        return dict(reg_qubits=r, thread_qubits=t, low_qubits=min(5, t + 1), plain=0, jit=0)
    hbm = 0.0
    for c, n, _, _ in items:
        p = qsv.sv_plan_info(c, layer_begin=1, opts=batch_opts(n))["n_passes"]
        hbm += (16.0 * p - 8.0) * (1 << n)
    achieved = hbm / tb / 1e9
    line = {
        "metric": METRIC, "value": au / tb, "unit": "amplitude-updates/s", "n_gpus": 1,
        "steps": a.steps, "warmup": 1, "ms_per_step": tb * 1e3, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBPS, "traffic": None,
                     "kernel": "whole batch graph (compiled and generic passes of all 512 circuits)",
                     "bytes_per_run": hbm},
        "config": {"workload": "uneven", "circuits": len(items), "n_range": [14, 26],
                   "depth_range": [8, 24], "state_bytes": sum(8 << n for _, n, _, _ in items),
                   "mode": "batched: one hipGraph launch; states of 2^21 amplitudes or more with compiled kernels of their own plan on the tile shape tuned for their size class, smaller ones one generic kernel per pass round"},
        "unbatched": {"value": au / tu, "ms_per_step": tu * 1e3,
                      "mode": "one sv_simulate per circuit with the batch's per-circuit options "
                              "(compiled kernels on the class-tuned tile from 2^21 amplitudes, "
                              "generic kernel below), each gathering its m amplitudes (each call "
                              "range-checks its bitstrings and waits for the stream first)",
                      "sweeps_only_ms": tus * 1e3},
        "plain": {"value": au / tp, "ms_per_step": tp * 1e3, "mode": "one kernel per gate"},
        "batched_vs_unbatched": tu / tb, "batched_vs_plain": tp / tb, "setup_s": setup_s,
        "caches": _caches(),
        "class_tuning": {"s": tune_s, "tiles": {str(n): [t["reg_qubits"], t["thread_qubits"], t["low_qubits"]]
                                                 for n, t in sorted(class_tiles.items())}},
        "scaled_error": {"checked": len(errs), "max": max(errs) if errs else None,
                         "median": float(np.median(errs)) if errs else None, "per_class": per_class},
    }
    print(json.dumps(line))


def bench_precision(a):
    """Precision form: 34 qubits (6x6 lattice minus two corners, depth 30,
    128 GiB complex64 state).  Runs the tuned fused sweep, the same circuit
    as forced dense 2^6 x 2^6 blocks on FP32 matrix cores, and the complex128
    instantiation of the compiled passes as reference; reports time, the
    matrix-core rate of the dense run and max |delta amp| of both FP32 runs
    against the FP64 run on 4096 sampled bitstrings, plus the FP64 norm."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    name = "6x6m2-d30"
    spec = workloads.WORKLOADS[name]
    n = spec["n"]
    dev = torch.device("cuda:0")
    pres = workloads.present_mask(spec)
    c = qsv.circuit_create(spec["rows"], spec["cols"], pres, spec["depth"], spec["seed"])
    n_gates = c.info()[2]
    xs = workloads.bitstrings(n, 4096, workloads.BITSTRING_SEED_BASE + 3)
    bits = torch.from_numpy(xs.view(np.int64)).to(dev)
    out32 = torch.empty(xs.size, dtype=torch.complex128, device=dev)
    outd = torch.empty(xs.size, dtype=torch.complex128, device=dev)
    out64 = torch.empty(xs.size, dtype=torch.complex128, device=dev)
    nrm = torch.zeros(1, dtype=torch.float64, device=dev)
    amps = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    ws = qsv.alloc_workspace(c, 1)
    t0 = time.perf_counter()
    tuned, _ = qsv.sv_tune(amps, c, layer_begin=1, workspace=ws)
    tune_s = time.perf_counter() - t0
    passes = qsv.sv_plan_info(c, layer_begin=1)["n_passes"]

    def fused():
        qsv.sv_simulate(amps, c, init_kind=qsv.INIT_PLUS, layer_begin=1, norm_out=nrm,
                        bitstrings=bits, amps_out=out32, c128=True, workspace=ws)
    fused()
    tf = _time_graph(fused, a.steps)
    norm32 = nrm.item()
    # forced dense blocks on matrix cores
    k = a.dense_k
    qsv.sv_init(amps, n, qsv.INIT_PLUS)
    blocks = qsv.sv_apply_dense(amps, c, k, layer_begin=1)  # builds the block plan
    torch.cuda.synchronize()

    def dense():
        qsv.sv_init(amps, n, qsv.INIT_PLUS)
        qsv.sv_apply_dense(amps, c, k, layer_begin=1)
        qsv.sv_amplitudes(amps, n, bits, outd, c128=True)
    td = _time_graph(dense, 1)
    del amps, ws
    torch.cuda.empty_cache()
    # complex128 reference (256 GiB)
    ref = torch.empty(1 << n, dtype=torch.complex128, device=dev)
    qsv.sv_simulate_c128(ref, c, init_kind=qsv.INIT_PLUS, layer_begin=1, norm_out=nrm,
                         bitstrings=bits, amps_out=out64)
    torch.cuda.synchronize()
    t64 = time.perf_counter()
    qsv.sv_simulate_c128(ref, c, init_kind=qsv.INIT_PLUS, layer_begin=1, norm_out=nrm,
                         bitstrings=bits, amps_out=out64)
    torch.cuda.synchronize()
    t64 = time.perf_counter() - t64
    norm64 = nrm.item()
    del ref
    torch.cuda.empty_cache()
    r64 = out64.cpu().numpy()
    d32 = float(np.max(np.abs(out32.cpu().numpy() - r64)))
    dd = float(np.max(np.abs(outd.cpu().numpy() - r64)))
    flops = blocks * 8.0 * (1 << k) * (1 << n)
    line = {
        "metric": METRIC, "value": n_gates * float(1 << n) / tf, "unit": "amplitude-updates/s",
        "n_gpus": 1, "steps": a.steps, "warmup": 1, "ms_per_step": tf * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": name, "mode": "precision", "n_qubits": n, "depth": spec["depth"],
                   "gates": n_gates, "passes": passes, "tile": tuned, "autotune_s": tune_s},
        "dense": {"k": k, "blocks": blocks, "ms": td * 1e3,
                  "value": n_gates * float(1 << n) / td,
                  "mfma_tflops": flops / td / 1e12, "mfma_peak_tflops": 157.3,
                  "mfma_frac": flops / td / 1e12 / 157.3,
                  "hbm_gbps": blocks * 16.0 * (1 << n) / td / 1e9},
        "fp64_reference": {"ms": t64 * 1e3, "norm": norm64},
        "error_vs_fp64": {"fused_max_abs": d32, "fused_scaled": d32 * 2 ** (n / 2),
                          "dense_max_abs": dd, "dense_scaled": dd * 2 ** (n / 2),
                          "sampled": int(xs.size)},
        "norm_fp64_of_f32_state": norm32, "norm_drift": abs(norm32 - 1.0),
    }
    print(json.dumps(line))


def bench_task2(a):
    """Task-2 amplitudes of the 30-qubit workload (5x6, depth 20) from two
    half-depth sweeps: |psi> = layers 1..10 on |+> once, then per bitstring x
    |phi> = (layers 11..20)^dagger |x> and <phi|psi> in FP64 (Section 2.2),
    accumulated by the adjoint sweep's last pass (sv_simulate_dot).  Reports
    time per amplitude, the two-step form (store phi, then sv_inner_product)
    and the error against the stored oracle amplitudes."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    name = "5x6-d20"
    spec = dict(workloads.WORKLOADS[name])
    n = spec["n"]
    dev = torch.device("cuda:0")
    pres = workloads.present_mask(spec)
    c = qsv.circuit_create(spec["rows"], spec["cols"], pres, spec["depth"], spec["seed"])
    inv = qsv.circuit_inverse(c)
    gates = c.gates()
    top = int(max(int(g["layer"]) for g in gates))
    h = 11
    g1 = sum(1 for g in gates if 1 <= int(g["layer"]) < h)
    g2 = sum(1 for g in gates if int(g["layer"]) >= h)
    xs, ref = golden(name)
    m = min(a.count, 64) if a.count else 16
    xs, ref = xs[:m], ref[:m]
    psi = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    phi = torch.empty_like(psi)
    dot = torch.zeros(2, dtype=torch.float64, device=dev)
    qsv.sv_tune(psi, c, layer_begin=1, layer_end=h)
    qsv.sv_tune(phi, inv, layer_begin=0, layer_end=top - h + 1)

    def forward():
        qsv.sv_simulate(psi, c, init_kind=qsv.INIT_PLUS, layer_begin=1, layer_end=h)

    def amplitude(x):
        # adjoint half from |x>, inner product accumulated by its last pass
        qsv.sv_simulate_dot(phi, inv, psi, dot, init_kind=qsv.INIT_BASIS, basis=int(x), layer_begin=0,
                            layer_end=top - h + 1)

    def amplitude_two_step(x):
        qsv.sv_simulate(phi, inv, init_kind=qsv.INIT_BASIS, basis=int(x), layer_begin=0,
                        layer_end=top - h + 1)
        qsv.sv_inner_product(phi, psi, n, dot)

    forward()
    amplitude(xs[0])
    amplitude_two_step(xs[0])
    t_fwd = _time_graph(forward, 3)
    forward()

    def run(fn):
        got = []
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for x in xs:
            fn(x)
            d = dot.cpu().numpy()  # synchronises: one amplitude at a time
            got.append(complex(d[0], d[1]))
        return (time.perf_counter() - t0) / len(xs), np.array(got)
    t_two, got_two = run(amplitude_two_step)
    t_amp, got = run(amplitude)
    err = float(np.max(np.abs(got - ref)))
    # all m amplitudes at once: the second half swept forward from psi, its
    # last pass sampled at the m bitstrings (only the tiles holding them)
    smp = qsv.sv_sampler_create(c, xs, layer_begin=h)
    samp = torch.empty(len(xs), dtype=torch.complex64, device=dev)
    qsv.sv_sampler_run(smp, psi, phi, samp)
    t_smp = _time_graph(lambda: qsv.sv_sampler_run(smp, psi, phi, samp), 5)
    err_smp = float(np.max(np.abs(samp.cpu().numpy() - ref)))
    total = t_fwd + t_amp * len(xs)
    line = {
        "metric": METRIC, "value": (g1 + g2 * len(xs)) * float(1 << n) / total,
        "unit": "amplitude-updates/s", "n_gpus": 1, "steps": len(xs), "warmup": 1,
        "ms_per_step": t_amp * 1e3, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "task2-5x6-d20", "n_qubits": n, "split_layer": h,
                   "gates_forward": g1, "gates_adjoint": g2, "amplitudes": len(xs)},
        "forward_half_ms": t_fwd * 1e3, "ms_per_amplitude": t_amp * 1e3,
        "two_step": {"ms_per_amplitude": t_two * 1e3, "mode": "adjoint sweep stored, then sv_inner_product",
                     "max_abs_diff_vs_fused": float(np.max(np.abs(got - got_two)))},
        "forward_sampled": {"ms_all_amplitudes": t_smp * 1e3, "amplitudes": len(xs),
                            "mode": "second half swept forward from the first, last pass sampled",
                            "max_abs_err": err_smp},
        "error": {"max_abs": err, "scaled": err * 2 ** (n / 2),
                  "vs": "complex128 oracle amplitudes (stored)"},
    }
    print(json.dumps(line))


def bench_combine(a):
    """Full-state combine of a cut circuit on matrix cores: the 30-qubit 5x6
    depth-16 circuit cut after column 2 (15 | 15 qubits, 1024 branch pairs).
    Times the batched branch sweeps of both halves and the complex GEMM
    Psi = A B^T (2^15 x 2^15 x 1024) with FP64 products and sums (and the
    FP32-accumulating option), reports each GEMM's matrix-core rate against
    its dtype's peak, the error against the stored oracle amplitudes, and the
    direct full-state sweep of the same circuit for comparison."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    name = "5x6-d16"
    spec = dict(workloads.WORKLOADS[name])
    n = spec["n"]
    dev = torch.device("cuda:0")
    pres = workloads.present_mask(spec)
    c = qsv.circuit_create(spec["rows"], spec["cols"], pres, spec["depth"], spec["seed"])
    mask = workloads.column_cut_mask(spec["rows"], spec["cols"], 2)
    ha, hb, ceff, folded = qsv.circuit_split(c, mask)
    na = bin(mask).count("1")
    nb_ = n - na
    nbr = 1 << ceff
    A = torch.empty(nbr, 1 << na, dtype=torch.complex64, device=dev)
    B = torch.empty(nbr, 1 << nb_, dtype=torch.complex64, device=dev)
    batch = qsv.sv_batch_create([ha] * nbr + [hb] * nbr, list(range(nbr)) * 2)
    states = [A[i] for i in range(nbr)] + [B[i] for i in range(nbr)]
    out = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    fa = [x for x, _ in folded]
    fb = [y for _, y in folded]

    def branches():
        qsv.sv_batch_run(batch, states, init_plus=True)

    def gemm():
        qsv.sv_branch_combine_full(A, B, nbr, na, nb_, mask, fa, fb, out)

    def gemm32():
        qsv.sv_branch_combine_full(A, B, nbr, na, nb_, mask, fa, fb, out, flags=qsv.COMBINE_FP32)

    xs, ref = golden(name)
    idx = torch.from_numpy(xs.view(np.int64)).to(dev)
    branches()
    gemm32()
    t_gemm32 = _time_graph(gemm32, 5)
    err32 = float(np.max(np.abs(out[idx].cpu().numpy() - ref)))
    gemm()
    t_br = _time_graph(branches, 5)
    t_gemm = _time_graph(gemm, 5)
    got = out[idx].cpu().numpy()
    err = float(np.max(np.abs(got - ref)))
    # direct sweep of the unsplit circuit
    amps = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    qsv.sv_tune(amps, c, layer_begin=1)

    def direct():
        qsv.sv_simulate(amps, c, init_kind=qsv.INIT_PLUS, layer_begin=1)
    direct()
    t_dir = _time_graph(direct, 5)
    flops = 8.0 * nbr * float(1 << n)
    g = c.info()[2]
    total = t_br + t_gemm
    line = {
        "metric": METRIC, "value": g * float(1 << n) / total, "unit": "amplitude-updates/s",
        "n_gpus": 1, "steps": 5, "warmup": 1, "ms_per_step": total * 1e3, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "combine-5x6-d16", "n_qubits": n, "halves": [na, nb_],
                   "branch_pairs": nbr, "folded": len(folded)},
        "branch_sweeps_ms": t_br * 1e3,
        "combine_gemm": {"ms": t_gemm * 1e3, "tflops": flops / t_gemm / 1e12, "peak_tflops": 78.6,
                         "frac": flops / t_gemm / 1e12 / 78.6, "bound": "mfma",
                         "precision": "FP64 products and sums (v_mfma_f64_16x16x4f64), complex64 output"},
        "combine_gemm_fp32": {"ms": t_gemm32 * 1e3, "tflops": flops / t_gemm32 / 1e12, "peak_tflops": 157.3,
                              "frac": flops / t_gemm32 / 1e12 / 157.3, "bound": "mfma",
                              "precision": "FP32 accumulation (option)", "max_abs_err": err32},
        "direct_sweep_ms": t_dir * 1e3,
        "error": {"max_abs": err, "scaled": err * 2 ** (n / 2), "vs": "complex128 oracle, 1024 sampled"},
    }
    print(json.dumps(line))


def bench_partition(a):
    """Complete 30-qubit state (5x6, depth 20) through the three-part
    partition of Section 2.1: Algorithm 1 plans the lines (initial cut after
    row 1); one sv_partition_simulate call runs every branch state of parts A
    and B in a batch, the combine GEMMs (one per value of the selector
    qubits) and the part-C sweep.  Reports the time per complete state, the
    error against the stored oracle amplitudes, and the direct sweep of the
    same circuit for comparison."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    name = "5x6-d20"
    spec = dict(workloads.WORKLOADS[name])
    n = spec["n"]
    dev = torch.device("cuda:0")
    pres = workloads.present_mask(spec)
    c = qsv.circuit_create(spec["rows"], spec["cols"], pres, spec["depth"], spec["seed"])
    t0 = time.perf_counter()
    p = qsv.circuit_partition_plan(c, spec["rows"], spec["cols"], pres, a.r0, a.max_move)
    t_plan = time.perf_counter() - t0
    info = qsv.circuit_partition_info(p)
    ws_bytes = qsv.sv_partition_workspace_bytes(p)
    ws = torch.empty(ws_bytes // 8, dtype=torch.complex64, device=dev)
    out = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    _, _, part_c, _, _ = qsv.circuit_partition_parts(p)
    qsv.sv_tune(out, part_c)  # remembered for the part-C circuit's content

    def run():
        qsv.sv_partition_simulate(p, ws, ws_bytes, out)
    t0 = time.perf_counter()
    run()
    torch.cuda.synchronize()
    t_first = time.perf_counter() - t0
    for _ in range(a.warmup):
        run()
    t_step = _time_graph(run, a.steps)
    xs, ref = golden(name)
    got = out[torch.from_numpy(xs.view(np.int64)).to(dev)].cpu().numpy()
    err = float(np.max(np.abs(got - ref)))
    nrm = torch.zeros(1, dtype=torch.float64, device=dev)
    qsv.sv_norm_fp64(out, n, nrm)
    del ws
    torch.cuda.empty_cache()
    amps = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    qsv.sv_tune(amps, c, layer_begin=1)

    def direct():
        qsv.sv_simulate(amps, c, init_kind=qsv.INIT_PLUS, layer_begin=1)
    direct()
    t_dir = _time_graph(direct, 5)
    g = c.info()[2]
    gemm_flops = 8.0 * float(1 << n) * float(1 << info["explicit_bits"])
    line = {
        "metric": METRIC, "value": g * float(1 << n) / t_step, "unit": "amplitude-updates/s",
        "n_gpus": 1, "steps": a.steps, "warmup": a.warmup, "ms_per_step": t_step * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "partition-5x6-d20", "n_qubits": n, "r0": a.r0, "max_move": a.max_move,
                   "scheme": {k: info[k] for k in ("t_s", "n_a", "n_b", "n_c", "cuts", "explicit_bits",
                                                   "sel_a", "sel_b", "folded", "f", "g",
                                                   "branches_a", "branches_b")}},
        "plan_ms": t_plan * 1e3, "first_call_s": t_first, "workspace_bytes": ws_bytes,
        "combine_gemm_flop": gemm_flops, "part_c_gates": int(part_c.info()[2]),
        "direct_sweep_ms": t_dir * 1e3,
        "error": {"max_abs": err, "scaled": err * 2 ** (n / 2), "vs": "complex128 oracle, 4096 sampled"},
        "norm_fp64": nrm.item(),
    }
    print(json.dumps(line))


def _small_tile_opts(c):
    """Options of the smallest whole-wave tile that plans the circuit into one
    pass (compiled kernels), or None."""
    from paper_1804_04797_amd import qsv
    for shape in ((3, 6, 1), (4, 6, 1), (4, 6, 2), (4, 7, 1), (5, 7, 1), (5, 8, 1)):
        o = dict(reg_qubits=shape[0], thread_qubits=shape[1], low_qubits=shape[2], plain=0, jit=1)
        if shape[0] + shape[1] <= c.n and qsv.sv_plan_info(c, 0, -1, o)["n_passes"] == 1:
            return o
    return None


def _stage_tree(h, xs, m, bufs, dev, merge=True, tune=True):
    """Every branch of the split half h as a tree over its branch stages
    (circuit_branch_stage): stage [0, 1) from |+> once, then level by level
    each child runs its stage from the parent state.  merge: the deepest
    levels whose joint stage plans into one pass form the leaves; otherwise
    every level is its own.  The leaves run their stage with the sampler
    (only the tiles holding the m bitstrings xs, on the smallest tile that
    plans it into one pass, all siblings in one launch).  Going up from the
    leaves, a level whose children read it only at a small part of its state
    runs as a tile sampler that computes just those tiles.  Returns (seconds
    per tree, leaf table [2^c_eff * m], description)."""
    import torch
    from paper_1804_04797_amd import qsv
    levels = qsv.circuit_branch_levels(h)
    L = len(levels)
    nbr = 1 << sum(bin(x).count("1") for x in levels)
    j = L
    while merge and j > 1 and qsv.sv_plan_info(qsv.circuit_branch_stage(h, j - 1, -1))["n_passes"] <= 1:
        j -= 1
    ranges = [(0, 1)] + [(k, k + 1) for k in range(1, j)] + [(j, L + 1)]
    stages = [qsv.circuit_branch_stage(h, a, b if b <= L else -1) for a, b in ranges]
    sbits = [[]] + [[b for b in range(64) if (sum(levels[k - 1] for k in range(a, e)) >> b) & 1]
                    for a, e in ranges[1:]]
    passes = [qsv.sv_plan_info(st, 1 if i == 0 else 0)["n_passes"] for i, st in enumerate(stages)]
    tab = torch.zeros(nbr * m, dtype=torch.complex64, device=dev)
    # compiled pass kernels also below 24 qubits (the generic kernel is the
    # default there)
    jit = dict(jit=1)
    leaf_opts = _small_tile_opts(stages[-1]) or jit
    sampler = qsv.sv_sampler_create(stages[-1], xs, layer_begin=0, opts=leaf_opts)
    # tile samplers for the levels above, as long as the level below reads a
    # small part of the state in one pass
    tiles = {}
    child = sampler if "reg_qubits" in leaf_opts else None
    for t in range(len(ranges) - 2, 0, -1):
        if child is None:
            break
        need = qsv.sv_sampler_inputs(child)
        # the default tile when it holds the stage in one pass (whole
        # workgroups of 4-8 waves run a tile list faster than one-wave tiles),
        # else the smallest one-pass tile
        o = jit if qsv.sv_plan_info(stages[t], 0, -1, jit)["n_passes"] == 1 else _small_tile_opts(stages[t])
        if o is None or need.size * 4 > (1 << h.n):
            break
        tiles[t] = qsv.sv_sampler_create_tiles(stages[t], need, layer_begin=0, opts=o)
        child = tiles[t]
    stage_out = torch.empty((1 << len(sbits[-1])) * m, dtype=torch.complex64, device=dev)
    # the root stage is a full sweep of the state: autotuned (setup) when the
    # compiled kernels are the default
    root_opts = jit
    if h.n >= 24:
        if tune:
            qsv.sv_tune(bufs[0], stages[0], layer_begin=1)
        root_opts = None
        passes[0] = qsv.sv_plan_info(stages[0], 1)["n_passes"]
    leaf_mask = sum(1 << b for b in sbits[-1])
    rows = {}
    calls = [0]
    work = bufs[len(ranges) - 1]  # the leaves' work buffer, never a tile sampler's src or target

    def tree():
        qsv.sv_simulate(bufs[0], stages[0], init_kind=qsv.INIT_PLUS, layer_begin=1, opts=root_opts)

        def rec(t, parent, prefix):
            brs = []
            for v in range(1 << len(sbits[t])):
                br = prefix
                for i, b in enumerate(sbits[t]):
                    br |= ((v >> i) & 1) << b
                brs.append(br)
            if t == len(ranges) - 1:
                # the sibling leaves in one launch; their rows of the table
                # are written in branch order through a staging table
                calls[0] += 1
                qsv.sv_sampler_run_subtree(sampler, parent, work, stage_out[:len(brs) * m], prefix, leaf_mask)
                if prefix not in rows:
                    rows[prefix] = torch.as_tensor(brs, device=dev)  # first (untimed) run only
                tab.view(nbr, m).index_copy_(0, rows[prefix], stage_out[:len(brs) * m].view(len(brs), m))
                return
            for br in brs:
                calls[0] += 1
                if t in tiles:
                    qsv.sv_sampler_run(tiles[t], parent, work, bufs[t], branch=br)
                else:
                    qsv.sv_apply_fused_from(parent, bufs[t], stages[t], branch=br, opts=jit)
                rec(t + 1, bufs[t], br)
        rec(1, bufs[0], 0)
    tree()
    torch.cuda.synchronize()
    calls[0] = 0
    sec = _time_graph(tree, 3)
    launches = calls[0] // 3
    # the same tree captured once into a graph (every launch of the tree,
    # the table scatter included) and replayed: checked against the eager
    # table on every replay, with eager work between the replays
    eager_tab = tab.clone()
    graph = {"ms": None}
    try:
        g = torch.cuda.CUDAGraph()
        cs = torch.cuda.Stream()
        cs.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=cs):
            tree()
        torch.cuda.synchronize()
        same = True
        for _ in range(3):
            tab.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            same = same and torch.equal(tab, eager_tab)
        graph = {"ms": _time_graph(g.replay, 3) * 1e3, "replays_identical_to_eager": same}
        del g
        if not same:
            raise RuntimeError("graph replay differs from the eager tree")
    except RuntimeError as ex:  # capture or replay failed: the eager tree stands
        graph["error"] = str(ex)[:200]
        tab.copy_(eager_tab)
    torch.cuda.synchronize()
    eager_sec = sec
    if graph["ms"] is not None and graph.get("replays_identical_to_eager"):
        sec = min(sec, graph["ms"] * 1e-3)
    info = {"eager_ms": eager_sec * 1e3, "graph": graph,
            "stage_levels": [list(r) for r in ranges], "stage_gates": [st.info()[2] for st in stages],
            "stage_passes": passes,
            "tree_states": [1] + [1 << sum(len(b) for b in sbits[1:k + 1]) for k in range(1, len(ranges))],
            "launch_groups": launches,
            "leaf_tile": [leaf_opts["reg_qubits"], leaf_opts["thread_qubits"]] if "reg_qubits" in leaf_opts
            else "default",
            "tile_sampled_levels": sorted(tiles)}
    return sec, tab, info


def bench_split(a):
    """Batched form: 49 qubits (7x7, depth 16) cut after column 3 into a
    28-qubit and a 21-qubit half; 11 cut CZs -> 2048 branch pairs, 3 final
    crossings folded into a sign.  The 28-qubit half (2 GiB per branch) runs
    as a tree over its branch stages: the gates that depend on no branch bit
    once, each later stage once per value of the branch bits fixed before its
    end, the leaves' stage by the sampler (only the tiles holding the sampled
    bitstrings); all 2048 leaves timed.  Comparators: the prefix tree split at
    the cut layers (every gate after a cut runs once per child), batches of
    --wave independent branches (--a-waves batches timed, all 2048 projected)
    and one sv_simulate per branch (same sample).  The 21-qubit half: all 2048
    branches in one batch (one graph launch) and its stage tree; the faster
    counts.  FP64 combine over 2048 x 1024."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads
    spec = workloads.WORKLOADS["7x7-d16"]
    dev = torch.device("cuda:0")
    c = qsv.circuit_create(7, 7, None, spec["depth"], spec["seed"])
    mask = workloads.column_cut_mask(7, 7, 3)
    ha, hb, ceff, folded = qsv.circuit_split(c, mask)
    na, nb_ = ha.n, hb.n
    nbr = 1 << ceff
    m = 1024
    xs = workloads.bitstrings(49, m, workloads.BITSTRING_SEED_BASE + 4)
    qa = [q for q in range(49) if (mask >> q) & 1]
    qb = [q for q in range(49) if not (mask >> q) & 1]

    def sub(x, qs):
        v = 0
        for i, q in enumerate(qs):
            v |= ((x >> q) & 1) << i
        return v
    xa = np.array([sub(int(x), qa) for x in xs], np.uint64)
    xb = np.array([sub(int(x), qb) for x in xs], np.uint64)
    sign = np.array([(-1) ** sum((int(x) >> p) & (int(x) >> q) & 1 for p, q in folded) for x in xs],
                    np.int8)
    ga, gb = ha.info()[2], hb.info()[2]
    # 21-qubit half: all branches, one batch
    bstates = [torch.empty(1 << nb_, dtype=torch.complex64, device=dev) for _ in range(nbr)]
    btab = torch.empty(nbr * m, dtype=torch.complex64, device=dev)
    bbits = torch.from_numpy(np.tile(xb, nbr).view(np.int64)).to(dev)
    bb = qsv.sv_batch_create([hb] * nbr, list(range(nbr)))
    qsv.sv_batch_run(bb, bstates, init_plus=True, bitstrings=bbits, m=m, amp_table=btab)
    tB = _time_graph(lambda: qsv.sv_batch_run(bb, bstates, init_plus=True, bitstrings=bbits, m=m,
                                              amp_table=btab), 3)
    # 28-qubit half: waves of branches
    W = a.wave
    atab = torch.zeros(nbr * m, dtype=torch.complex64, device=dev)
    astates = [torch.empty(1 << na, dtype=torch.complex64, device=dev) for _ in range(W)]
    abits = torch.from_numpy(np.tile(xa, W).view(np.int64)).to(dev)
    waves = []
    for wv in range(a.a_waves):
        brs = list(range(wv * W, (wv + 1) * W))
        waves.append((qsv.sv_batch_create([ha] * W, brs), wv))
    b0, _ = waves[0]
    qsv.sv_batch_run(b0, astates, init_plus=True, bitstrings=abits, m=m, amp_table=atab[:W * m])
    torch.cuda.synchronize()

    def run_waves():
        for bw, wv in waves:
            qsv.sv_batch_run(bw, astates, init_plus=True, bitstrings=abits, m=m,
                             amp_table=atab[wv * W * m:(wv + 1) * W * m])
    run_waves()
    tA = _time_graph(run_waves, 1)
    sampleA = W * a.a_waves
    tA_full = tA * nbr / sampleA
    # combine (full size)
    out = torch.empty(m, dtype=torch.complex128, device=dev)
    sg = torch.from_numpy(sign).to(dev)
    tC = _time_graph(lambda: qsv.sv_branch_combine(atab.view(nbr, m), btab.view(nbr, m), nbr, m,
                                                   sg, out), 5)
    # unbatched comparator on the same sample (skipped with --no-plain)
    tUA = tUB = None
    xat = torch.from_numpy(xa.view(np.int64)).to(dev)
    if not a.no_plain:
        one = torch.empty(1 << na, dtype=torch.complex64, device=dev)
        o1 = torch.empty(m, dtype=torch.complex64, device=dev)
        xbt = torch.from_numpy(xb.view(np.int64)).to(dev)

        def unb_a():
            for br in range(sampleA):
                qsv.sv_simulate(one, ha, branch=br, init_kind=qsv.INIT_PLUS, layer_begin=1,
                                bitstrings=xat, amps_out=o1)
        unb_a()
        tUA = _time_graph(unb_a, 1) * nbr / sampleA
        onb = torch.empty(1 << nb_, dtype=torch.complex64, device=dev)

        def unb_b():
            for br in range(nbr):
                qsv.sv_simulate(onb, hb, branch=br, init_kind=qsv.INIT_PLUS, layer_begin=1,
                                bitstrings=xbt, amps_out=o1)
        unb_b()
        tUB = _time_graph(unb_b, 1)
    # 28-qubit half as a branch tree with shared prefixes: the state at each
    # cut layer is computed once and each child continues from it
    # (sv_apply_fused_from), every leaf's sampled amplitudes gathered; all
    # 2048 leaves are timed (no projection)
    del astates
    torch.cuda.empty_cache()
    g_a = ha.gates()
    cut = sorted({(int(x["layer"]), int(x["arg"])) for x in g_a if int(x["kind"]) in (qsv.KIND["PB"], qsv.KIND["ZB"])})
    layers = sorted({l for l, _ in cut})
    bits_at = {l: [b for l2, b in cut if l2 == l] for l in layers}
    tbufs = [torch.empty(1 << na, dtype=torch.complex64, device=dev) for _ in range(len(layers) + 1)]
    ttab = torch.zeros(nbr * m, dtype=torch.complex64, device=dev)
    calls = [0]
    # leaves: only the last pass's tiles that hold the sampled bitstrings
    leaf_sampler = qsv.sv_sampler_create(ha, xa, layer_begin=layers[-1])

    def tree():
        qsv.sv_simulate(tbufs[0], ha, init_kind=qsv.INIT_PLUS, layer_begin=1, layer_end=layers[0])

        def rec(level, parent, prefix):
            lb = layers[level - 1]
            le = layers[level] if level < len(layers) else -1
            for v in range(1 << len(bits_at[lb])):
                br = prefix
                for i, b in enumerate(bits_at[lb]):
                    br |= ((v >> i) & 1) << b
                calls[0] += 1
                if level == len(layers):
                    qsv.sv_sampler_run(leaf_sampler, parent, tbufs[level], ttab[br * m:(br + 1) * m], branch=br)
                else:
                    qsv.sv_apply_fused_from(parent, tbufs[level], ha, branch=br, layer_begin=lb, layer_end=le)
                    rec(level + 1, tbufs[level], br)
        rec(1, tbufs[0], 0)
    tL, layer_calls = None, None
    if not a.no_plain:  # the comparator (skipped with --no-plain)
        tree()
        torch.cuda.synchronize()
        calls[0] = 0
        tL = _time_graph(tree, 1)
        layer_calls = calls[0]
    # The same tree over branch stages (circuit_branch_stage): a gate runs at
    # the shallowest tree level that fixes every branch bit it depends on, so
    # the gates that commute past the cuts run once at the root; the deepest
    # levels whose stage is a single pass are merged into the leaves, whose
    # only pass is the sampled one.
    # both tree shapes (leaf levels merged or not); the faster one counts
    tT, stab, st_info = _stage_tree(ha, xa, m, tbufs, dev, merge=True)
    tT2, stab2, st_info2 = _stage_tree(ha, xa, m, tbufs, dev, merge=False, tune=False)
    other_shape_vs = float((stab2 - stab).abs().max().item())
    other_shape = dict(st_info2 if tT2 >= tT else st_info, ms=max(tT, tT2) * 1e3)
    if tT2 < tT:
        tT, stab, st_info = tT2, stab2, st_info2
    # the 21-qubit half the same way (2048 small leaves), against its batch
    bbufs = [torch.empty(1 << nb_, dtype=torch.complex64, device=dev) for _ in range(4)]
    tTB, stabB, st_infoB = _stage_tree(hb, xb, m, bbufs, dev, merge=True)
    tTB2, stabB2, st_infoB2 = _stage_tree(hb, xb, m, bbufs, dev, merge=False)
    if tTB2 < tTB:
        tTB, stabB, st_infoB = tTB2, stabB2, st_infoB2
    tree_b_vs_batch = float((stabB - btab).abs().max().item())
    # the trees' leaves agree with the batched branches of the sample and with each other
    tree_vs_batched = float((stab[:sampleA * m] - atab[:sampleA * m]).abs().max().item())
    stage_vs_layer_tree = float((stab - ttab).abs().max().item()) if tL is not None else None
    # leaves against independent full sweeps of the same branches
    tree_vs_direct = 0.0
    got = torch.empty(m, dtype=torch.complex64, device=dev)
    for br in (0, 1337, nbr - 1):
        qsv.sv_simulate(tbufs[-1], ha, branch=br, init_kind=qsv.INIT_PLUS, layer_begin=1)
        qsv.sv_amplitudes(tbufs[-1], na, xat, got)
        tree_vs_direct = max(tree_vs_direct, float((got - stab[br * m:(br + 1) * m]).abs().max().item()))
    outT = torch.empty(m, dtype=torch.complex128, device=dev)
    qsv.sv_branch_combine(stab.view(nbr, m), btab.view(nbr, m), nbr, m, sg, outT)
    combine_tree_vs_batched = None
    if sampleA == nbr:
        combine_tree_vs_batched = float((outT - out).abs().max().item())
    au = nbr * (ga * float(1 << na) + gb * float(1 << nb_))
    # the faster of the two measured forms of the 21-qubit half counts
    tBbest = min(tB, tTB)
    total = tT + tBbest + tC
    line = {
        "metric": METRIC, "value": au / total, "unit": "amplitude-updates/s", "n_gpus": 1,
        "steps": 1, "warmup": 1, "ms_per_step": total * 1e3, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "7x7-d16", "cut": "after column 3", "halves": [na, nb_],
                   "c_eff": ceff, "folded": len(folded), "branch_pairs": nbr,
                   "output_bitstrings": m, "wave": W,
                   "sample_28q_branches": sampleA},
        "half_28q": {"ms": tT * 1e3,
                     "mode": "branch tree over branch stages (each gate at the shallowest level that fixes "
                             "its branch bits), all 2048 leaves sampled (a leaf's only pass runs the tiles "
                             "holding the 1024 bitstrings)",
                     **st_info,
                     "other_tree_shape": other_shape,
                     "other_tree_shape_vs_max_abs": other_shape_vs,
                     "leaves_vs_batched_sample_max_abs": tree_vs_batched,
                     "leaves_vs_layer_tree_max_abs": stage_vs_layer_tree,
                     "layer_tree": {"ms": tL * 1e3 if tL is not None else None,
                                    "mode": "prefix tree split at the cut layers, "
                                                          "leaves sampled",
                                    "tree_levels": [1] + [1 << sum(len(bits_at[l]) for l in layers[:k + 1])
                                                          for k in range(len(layers))],
                                    "sweeps_from_parent": layer_calls},
                     "batched_waves_ms_projected_all": tA_full * 1e3, "batched_waves_ms_sample": tA * 1e3},
        "leaves_vs_direct_sweep_max_abs": tree_vs_direct,
        "half_21q": {"ms": tBbest * 1e3, "batch_ms": tB * 1e3,
                     "batch_mode": "all 2048 branches in one batch (one graph launch)",
                     "stage_tree_ms": tTB * 1e3, "stage_tree": st_infoB,
                     "stage_tree_vs_batch_max_abs": tree_b_vs_batch},
        "combine_ms": tC * 1e3,
        "batched_waves_total_ms_projected": (tA_full + tB + tC) * 1e3,
        "unbatched": {"ms_projected": (tUA + tUB + tC) * 1e3 if tUA is not None else None,
                      "value": au / (tUA + tUB + tC) if tUA is not None else None,
                      "mode": "one sv_simulate per branch (compiled passes)"},
        "batched_vs_unbatched": (tUA + tUB + tC) / total if tUA is not None else None,
    }
    print(json.dumps(line))


def _cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def bench_sweep(a, name, full=True):
    """One workload of the full-state sweep: autotune (setup), then the timed
    steps, the error against the complex128 reference, and (full=True) the
    unfused comparator, the streaming-copy ceiling and the CPU oracle."""
    import numpy as np
    import torch
    from paper_1804_04797_amd import qsv, workloads

    spec = dict(workloads.WORKLOADS[name])
    spec["name"] = name
    n = spec["n"]
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    opts = None
    if a.reg or a.thr or a.low:
        opts = dict(reg_qubits=a.reg, thread_qubits=a.thr, low_qubits=a.low, plain=0, jit=a.jit,
                    pass_forms=a.pass_forms)
    pres = workloads.present_mask(spec)

    if a.calibrate_copy:
        src = torch.ones(1 << 28, dtype=torch.float32, device=dev)  # 1 GiB
        dst = torch.empty_like(src)
        qsv.sv_stream_copy(src, dst, 1 << 30)
        torch.cuda.synchronize()
        del src, dst
    amps = torch.empty(1 << n, dtype=torch.complex64, device=dev)
    xs_np, ref = golden(name)
    if xs_np is None:
        xs_np = workloads.bitstrings(n, 4096, workloads.BITSTRING_SEED_BASE + {"6x6m2-d30": 3}.get(name, 2))
    xs = torch.from_numpy(xs_np.view(np.int64)).to(dev)
    out = torch.empty(xs_np.size, dtype=torch.complex128, device=dev)
    nrm = torch.zeros(1, dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream()
    c0 = qsv.circuit_create(spec["rows"], spec["cols"], pres, spec["depth"], spec["seed"])
    # one caller-owned workspace (second state buffer + partial sums), sized
    # for the options before tuning (the tuned shape fits it too)
    ws = qsv.alloc_workspace(c0, 1, -1, opts)

    ev = []

    def step(timed):
        c = qsv.circuit_create(spec["rows"], spec["cols"], pres, spec["depth"], spec["seed"])
        if timed:
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
        qsv.sv_simulate(amps, c, init_kind=qsv.INIT_PLUS, layer_begin=1, opts=opts, norm_out=nrm,
                        bitstrings=xs, amps_out=out, c128=True, workspace=ws)
        if timed:
            e1.record(stream)
            ev.append((e0, e1))
        return c

    tuned, tune_s = None, None
    if opts is None and not a.no_tune:
        # autotune once per circuit (setup, like kernel compilation): the
        # steps below call sv_simulate with opts=None and get the tuned shape
        t_tune = time.perf_counter()
        tuned, tuned_ms = qsv.sv_tune(amps, c0, layer_begin=1, workspace=ws)
        tune_s = time.perf_counter() - t_tune
        if a.jit:
            opts = dict(tuned, jit=a.jit)
    c = step(False)
    n_gates = c.info()[2]
    passes = qsv.sv_plan_info(c, layer_begin=1, opts=opts)["n_passes"]
    for _ in range(a.warmup):
        step(False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(a.steps):
        step(True)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms = (t1 - t0) * 1e3 / a.steps
    value = n_gates * float(1 << n) / (ms * 1e-3)

    # Dominant kernel: the fused pass.  The first pass generates |+>^n in
    # registers and only writes (8 bytes per amplitude); every later pass
    # reads and writes (16 bytes per amplitude).  The events bracket the
    # passes plus the tiny norm-partial sum and gather kernels.
    sweep_ms = sum(e0.elapsed_time(e1) for e0, e1 in ev) / len(ev)
    launch_ms = sweep_ms / passes
    sweep_bytes = (16.0 * passes - 8.0) * (1 << n)
    bytes_per_launch = sweep_bytes / passes
    achieved = bytes_per_launch / (launch_ms * 1e-3) / 1e9
    traffic = None
    shape = opts or tuned or {"reg_qubits": 0, "thread_qubits": 0, "low_qubits": 0}
    if a.traffic_json and os.path.exists(a.traffic_json):
        tj = json.load(open(a.traffic_json))
        t = tj.get(name)
        if (t and t.get("shape") == [shape["reg_qubits"], shape["thread_qubits"], shape["low_qubits"]]
                and t.get("pass_forms", shape.get("pass_forms")) == shape.get("pass_forms")
                and t.get("kernel_rev") == qsv.version()):
            traffic = t.get("bytes_per_launch")
    got = out.cpu().numpy()
    norm_drift = abs(nrm.item() - 1.0)

    plain = None
    if full and not a.no_plain:
        qsv.sv_init(amps, n, qsv.INIT_PLUS)
        qsv.sv_apply_plain(amps, c, layer_begin=1)
        torch.cuda.synchronize()
        tp0 = time.perf_counter()
        qsv.sv_init(amps, n, qsv.INIT_PLUS)
        qsv.sv_apply_plain(amps, c, layer_begin=1)
        qsv.sv_norm_fp64(amps, n, nrm)
        pout = torch.empty_like(out)
        qsv.sv_amplitudes(amps, n, xs, pout, c128=True)
        torch.cuda.synchronize()
        tp = time.perf_counter() - tp0
        plain = {"value": n_gates * float(1 << n) / tp, "ms_per_step": tp * 1e3,
                 "_out": pout.cpu().numpy(), "speedup_fused_vs_plain": (tp * 1e3) / ms}

    # measured streaming ceiling: sv_stream_copy of the state (the sweep's
    # 16-byte nontemporal accesses, one read and one write per amplitude)
    copy_gbps = None
    if full and n >= 24:
        dst = ws[:8 << n] if ws.numel() >= (8 << n) else torch.empty(8 << n, dtype=torch.uint8, device=dev)
        qsv.sv_stream_copy(amps, dst, 8 << n)
        cs = torch.cuda.current_stream()
        k0, k1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        k0.record(cs)
        for _ in range(5):
            qsv.sv_stream_copy(amps, dst, 8 << n)
        k1.record(cs)
        k1.synchronize()
        copy_gbps = 5 * 16.0 * (1 << n) / (k0.elapsed_time(k1) * 1e-3) / 1e9
        del dst
    del amps, ws
    torch.cuda.empty_cache()

    # error reference: the stored complex128 oracle amplitudes, or (states the
    # host cannot hold) the complex128 instantiation of the compiled passes
    if ref is not None:
        ref_kind = "complex128 oracle, 4096 sampled"
    else:
        r128 = torch.empty(1 << n, dtype=torch.complex128, device=dev)
        rout = torch.empty_like(out)
        qsv.sv_simulate_c128(r128, c, init_kind=qsv.INIT_PLUS, layer_begin=1, bitstrings=xs, amps_out=rout)
        torch.cuda.synchronize()
        ref = rout.cpu().numpy()
        del r128
        torch.cuda.empty_cache()
        ref_kind = "complex128 instantiation of the compiled passes on the device, 4096 sampled"
    d = float(np.max(np.abs(got - ref)))
    err = {"max_abs": d, "scaled": d * 2 ** (n / 2), "vs": ref_kind}
    if plain is not None:
        pd = float(np.max(np.abs(plain.pop("_out") - ref)))
        plain["max_abs_err"] = pd

    cpu = None
    if full and not a.no_cpu:
        cpu = cpu_baseline(spec, a.cpu_seconds)
        cpu["single_thread"] = cpu_single_thread(name, max(2.0, a.cpu_seconds / 3))
        cpu["cpu_model"] = _cpu_model()

    line = {
        "metric": METRIC, "value": value, "unit": "amplitude-updates/s", "n_gpus": 1,
        "steps": a.steps, "warmup": a.warmup, "ms_per_step": ms, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": name, "n_qubits": n, "lattice": f"{spec['rows']}x{spec['cols']}",
                   "absent_sites": [list(x) for x in spec["absent"]],
                   "depth": spec["depth"], "gates": n_gates, "passes": passes,
                   "sampled_bitstrings": int(xs_np.size),
                   "tile": opts or tuned or "default", "autotune_s": tune_s,
                   "steps_include": "create+plan+init+sweep+norm+gather"},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBPS, "traffic": traffic,
                     "copy_ceiling_GBps": copy_gbps,
                     "frac_of_copy_ceiling": achieved / copy_gbps if copy_gbps else None,
                     "kernel": "qsv_pass_* (compiled fused passes)", "launch_ms": launch_ms,
                     "bytes_per_launch": bytes_per_launch},
        "hbm_gbps_step": sweep_bytes / (ms * 1e-3) / 1e9,
        "error": err, "norm_drift": norm_drift,
        "plain": plain,
        "cpu_baseline": cpu,
        "caches": _caches(),
    }
    return line


def main():
    a = parse()
    if a.gpus != 1:
        print("bench.py runs on one GPU only: the library has no multi-GPU path "
              "(use --gpus 1)", file=sys.stderr)
        sys.exit(2)
    if a.cpu_probe > 0:  # child process of cpu_single_thread (no GPU use)
        from paper_1804_04797_amd import workloads
        spec = dict(workloads.WORKLOADS[a.workload])
        spec["name"] = a.workload
        print(json.dumps(cpu_baseline(spec, a.cpu_probe, max_qubits=30)))
        return
    if a.workload == "uneven":
        return bench_uneven(a)
    if a.workload == "precision":
        return bench_precision(a)
    if a.workload == "7x7-d16":
        return bench_split(a)
    if a.workload == "task2":
        return bench_task2(a)
    if a.workload == "combine":
        return bench_combine(a)
    if a.workload == "partition":
        return bench_partition(a)
    line = bench_sweep(a, a.workload, full=True)
    if a.secondary and a.secondary != a.workload:
        # the same sweep on a second workload (smaller state, stored oracle
        # amplitudes), reported beside the headline
        sec = bench_sweep(a, a.secondary, full=False)
        line["secondary"] = {k: sec[k] for k in ("value", "ms_per_step", "config", "roofline", "error",
                                                 "norm_drift", "hbm_gbps_step")}
    print(json.dumps(line))


if __name__ == "__main__":
    main()
