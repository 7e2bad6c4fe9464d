"""The work that programs built on the library have it do, as measurable cases.

Sizes follow the repository's own workloads (4x5 depth 10, 5x6 depth 20, the
5x6 depth-16 cut after column 2, 2048 branch pairs at 1024 sampled outputs,
uneven batches of 14-qubit and larger circuits) and ordinary values between
and below them.  Every call goes through paper_1804_04797_amd.qsv with default
options.  `exact` computes the same results in complex128 with plain torch
from this file's own generator of the circuit family.

Kinds of case:
  apply          a sweep over a state the program holds (in place, or from a
                 parent state into another buffer as branch trees do)
  simulate       a whole circuit in one call: start, sweep, FP64 norm, gather
  sample         amplitudes of a half sweep at given bitstrings from a stored state
  dense          the gates as 2^k x 2^k blocks on matrix cores
  branches       every branch state of both halves of a cut circuit, one batch
  uneven         independent circuits of different sizes, one batch
  combine        sampled amplitudes from the tables of both halves' branches
  combine_full   the complete state from all branch states of both halves
  reduce         FP64 norm or inner product of stored states
"""
import math
import random

import numpy as np
import torch

from paper_1804_04797_amd import qsv

DEV = "cuda"


def listed():
    return [
        # smallest sweep: a 16-qubit state updated in place; launches and latency count
        dict(name="apply_16q", kind="apply", n=16, rows=4, cols=4, depth=12, circuit=11, in_place=True),
        # the 4x5 depth-10 workload in one call from a basis state, 64 amplitudes read
        dict(name="simulate_20q", kind="simulate", n=20, rows=4, cols=5, depth=10, circuit=12, start="basis", m=64),
        # a ragged lattice, the largest size that does not compile its passes
        dict(name="simulate_23q", kind="simulate", n=23, rows=4, cols=6, depth=14, circuit=13, start="basis", m=256),
        # a child state of a branch tree: out of place from its parent, ragged lattice
        dict(name="apply_from_26q", kind="apply", n=26, rows=5, cols=6, depth=24, circuit=14, in_place=False),
        # the 5x6 depth-20 workload, 8 GiB state, as the benchmark's step runs it
        dict(name="simulate_30q", kind="simulate", n=30, rows=5, cols=6, depth=20, circuit=15, start="plus", m=4096),
        # Task-2 amplitudes of the second half sweep from the stored first half
        dict(name="sample_28q", kind="sample", n=28, rows=4, cols=7, depth=16, circuit=16, m=64),
        # dense gate sets on matrix cores
        dict(name="dense_24q", kind="dense", n=24, rows=4, cols=6, depth=8, circuit=17, k=6),
        # both halves of the 5x6 depth-16 cut: 2 x 1024 states of 15 qubits
        dict(name="branches_15q", kind="branches", rows=5, cols=6, after=2, depth=16, branches=1024),
        # independent circuits of 14..24 qubits, one graph, 16 amplitudes each
        dict(name="uneven_32", kind="uneven", count=32, lo=14, hi=24, circuit=18, m=16),
        # 2048 branch pairs at 1024 sampled outputs (the 49-qubit cut's table)
        dict(name="combine_2048", kind="combine", branches=2048, m=1024),
        # the complete 30-qubit state of the same cut: 2^15 x 2^15 x 1024
        dict(name="combine_full_30q", kind="combine_full", rows=5, cols=6, after=2, branches=1024),
        # an inner product of two stored 4 GiB states
        dict(name="inner_29q", kind="reduce", op="inner", n=29),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def lattice(n):
    rows = math.isqrt(n)
    return rows, -(-n // rows)


def draw(rng):
    kind = rng.choice(["apply", "simulate", "simulate", "sample", "dense", "branches", "uneven", "combine",
                       "combine_full", "reduce"])
    circuit = rng.randrange(1, 1 << 30)
    if kind == "apply":
        n = rng.randint(12, 28)
        rows, cols = lattice(n)
        return dict(kind=kind, n=n, rows=rows, cols=cols, depth=rng.randint(8, 24), circuit=circuit,
                    in_place=rng.random() < 0.5)
    if kind == "simulate":
        n = rng.randint(13, 29)
        rows, cols = lattice(n)
        return dict(kind=kind, n=n, rows=rows, cols=cols, depth=rng.randint(8, 24), circuit=circuit,
                    start=rng.choice(["plus", "basis"]), m=log_int(rng, 1, 4096))
    if kind == "sample":
        n = rng.randint(22, 29)
        rows, cols = lattice(n)
        return dict(kind=kind, n=n, rows=rows, cols=cols, depth=rng.randint(8, 20), circuit=circuit,
                    m=log_int(rng, 1, 1024))
    if kind == "dense":
        n = rng.randint(18, 25)
        rows, cols = lattice(n)
        return dict(kind=kind, n=n, rows=rows, cols=cols, depth=rng.randint(4, 10), circuit=circuit,
                    k=rng.randint(4, 7))
    if kind == "branches":
        rows, cols, after = rng.choice([(4, 6, 2), (5, 6, 2), (4, 7, 2), (4, 8, 3), (6, 4, 1), (5, 5, 2)])
        return dict(kind=kind, rows=rows, cols=cols, after=after, depth=rng.randint(10, 18),
                    branches=log_int(rng, 16, 1024 if rows * cols <= 30 else 512))
    if kind == "uneven":
        lo = rng.randint(12, 16)
        return dict(kind=kind, count=rng.randint(4, 40), lo=lo, hi=lo + rng.randint(3, 7), circuit=circuit,
                    m=log_int(rng, 1, 64))
    if kind == "combine":
        return dict(kind=kind, branches=log_int(rng, 8, 4096), m=log_int(rng, 1, 4096))
    if kind == "combine_full":
        rows, cols, after = rng.choice([(4, 4, 1), (3, 6, 2), (4, 5, 1), (4, 5, 2), (5, 5, 2), (4, 6, 2), (4, 7, 3),
                                        (5, 6, 2)])
        return dict(kind=kind, rows=rows, cols=cols, after=after, branches=log_int(rng, 2, 1000))
    return dict(kind=kind, op=rng.choice(["norm", "inner"]), n=rng.randint(10, 29))


# --- inputs ----------------------------------------------------------------


def generator(seed, stream=0):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1009 + stream) % (1 << 62))


def random_states(shape, norm, seed, stream=0):
    """Complex Gaussian amplitudes (what deep random circuits give), complex64."""
    out = torch.empty(shape, dtype=torch.complex64, device=DEV)
    torch.view_as_real(out).normal_(0.0, norm * math.sqrt(0.5), generator=generator(seed, stream))
    return out


def random_bits(n, m, seed):
    rng = random.Random(seed * 31 + 7)
    return [rng.randrange(1 << n) for _ in range(m)]


def present(case):
    sites = case["rows"] * case["cols"]
    return [1 if i < case.get("n", sites) else 0 for i in range(sites)]


def device_bits(xs):
    return torch.tensor(xs, dtype=torch.int64, device=DEV)


def make_circuit(case, seed=None):
    return qsv.circuit_create(case["rows"], case["cols"], present(case), case["depth"],
                              case["circuit"] if seed is None else seed)


def left_mask(case):
    """Qubits of columns 0..after of a full rows x cols lattice."""
    return sum(1 << (r * case["cols"] + c) for r in range(case["rows"]) for c in range(case["after"] + 1))


def halves(case):
    na = case["rows"] * (case["after"] + 1)
    return na, case["rows"] * case["cols"] - na


def uneven_items(case, seed):
    """(n, depth, circuit seed): a program compiles the large circuits once
    and brings new small ones."""
    rng = random.Random(case["circuit"])
    items = []
    for i in range(case["count"]):
        n, d, s = rng.randint(case["lo"], case["hi"]), rng.randint(8, 24), rng.randrange(1 << 60)
        items.append((n, d, s if n >= 21 else s ^ ((seed * 64 + i) & 0xFFFFFFFFFFFF)))
    return items


def folded_pairs(case):
    a = case["after"]
    left = [r * case["cols"] + a for r in range(0, case["rows"], 2)]
    return left, [q + 1 for q in left]


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind == "apply":
        n = case["n"]
        s["circuit"] = c = make_circuit(case)
        s["src"] = random_states(1 << n, 2.0 ** (-n / 2), seed)
        s["dst"] = s["src"] if case["in_place"] else torch.empty_like(s["src"])
        s["ws"] = qsv.alloc_workspace(c, 1, -1)
    elif kind == "simulate":
        n = case["n"]
        first = 0 if case["start"] == "basis" else 1
        s["circuit"] = c = make_circuit(case)
        s["basis"] = random_bits(n, 1, seed + 1)[0] if case["start"] == "basis" else 0
        s["bits"] = device_bits(random_bits(n, case["m"], seed))
        s["amps"] = torch.empty(1 << n, dtype=torch.complex64, device=DEV)
        s["out"] = torch.empty(case["m"], dtype=torch.complex128, device=DEV)
        s["norm"] = torch.empty(1, dtype=torch.float64, device=DEV)
        s["ws"] = qsv.alloc_workspace(c, first, -1)
    elif kind == "sample":
        n, half = case["n"], case["depth"] // 2
        s["circuit"] = c = make_circuit(case)
        s["sampler"] = qsv.sv_sampler_create(c, random_bits(n, case["m"], seed), layer_begin=half)
        s["src"] = random_states(1 << n, 2.0 ** (-n / 2), seed)
        s["work"] = torch.empty_like(s["src"])
        s["out"] = torch.empty(case["m"], dtype=torch.complex64, device=DEV)
        s["ws"] = qsv.alloc_workspace(c, half, -1)
    elif kind == "dense":
        n = case["n"]
        s["circuit"] = make_circuit(case)
        s["amps"] = random_states(1 << n, 2.0 ** (-n / 2), seed)
    elif kind == "branches":
        na, nb = halves(case)
        c = make_circuit(case, seed)
        ha, hb, cuts, _ = qsv.circuit_split(c, left_mask(case))
        k = case["branches"]
        ids = [b & ((1 << cuts) - 1) for b in range(k)]
        s["a"] = torch.empty(k, 1 << na, dtype=torch.complex64, device=DEV)
        s["b"] = torch.empty(k, 1 << nb, dtype=torch.complex64, device=DEV)
        s["where"] = [x.data_ptr() + 8 * i * x.stride(0) for x in (s["a"], s["b"]) for i in range(k)]
        s["batch"] = qsv.sv_batch_create([ha] * k + [hb] * k, ids * 2)
    elif kind == "uneven":
        items = uneven_items(case, seed)
        s["states"] = torch.empty(sum(1 << n for n, _, _ in items), dtype=torch.complex64, device=DEV)
        circuits, at = [], 0
        s["where"] = []
        for n, d, cs in items:
            rows, cols = lattice(n)
            circuits.append(make_circuit(dict(n=n, rows=rows, cols=cols, depth=d, circuit=cs)))
            s["where"].append(s["states"].data_ptr() + 8 * at)
            at += 1 << n
        s["bits"] = device_bits([x for i, (n, _, _) in enumerate(items) for x in random_bits(n, case["m"], seed * 64 + i)])
        s["table"] = torch.empty(len(items) * case["m"], dtype=torch.complex64, device=DEV)
        s["batch"] = qsv.sv_batch_create(circuits)
    elif kind == "combine":
        shape = (case["branches"], case["m"])
        s["a"] = random_states(shape, 2.0 ** -14, seed, 1)
        s["b"] = random_states(shape, 2.0 ** -10, seed, 2)
        s["sign"] = (1 - 2 * torch.randint(0, 2, (case["m"],), device=DEV, generator=generator(seed, 3))).to(torch.int8)
        s["out"] = torch.empty(case["m"], dtype=torch.complex128, device=DEV)
    elif kind == "combine_full":
        na, nb = halves(case)
        s["a"] = random_states((case["branches"], 1 << na), 2.0 ** (-na / 2), seed, 1)
        s["b"] = random_states((case["branches"], 1 << nb), 2.0 ** (-nb / 2), seed, 2)
        s["out"] = torch.empty(1 << (na + nb), dtype=torch.complex64, device=DEV)
        s["fold"] = [np.array(v, dtype=np.int32) for v in folded_pairs(case)]
    else:
        n = case["n"]
        s["a"] = random_states(1 << n, 2.0 ** (-n / 2), seed, 1)
        s["b"] = random_states(1 << n, 2.0 ** (-n / 2), seed, 2) if case["op"] == "inner" else None
        s["out"] = torch.empty(2 if case["op"] == "inner" else 1, dtype=torch.float64, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "apply":
        if case["in_place"]:
            qsv.sv_apply_fused(s["dst"], s["circuit"], layer_begin=1, workspace=s["ws"])
        else:
            qsv.sv_apply_fused_from(s["src"], s["dst"], s["circuit"], layer_begin=1, workspace=s["ws"])
        return s["dst"]
    if kind == "simulate":
        basis = case["start"] == "basis"
        qsv.sv_simulate(s["amps"], s["circuit"], init_kind=qsv.INIT_BASIS if basis else qsv.INIT_PLUS,
                        basis=s["basis"], layer_begin=0 if basis else 1, norm_out=s["norm"], bitstrings=s["bits"],
                        amps_out=s["out"], c128=True, workspace=s["ws"])
        return {"state": s["amps"], "norm": s["norm"], "amplitudes": s["out"]}
    if kind == "sample":
        qsv.sv_sampler_run(s["sampler"], s["src"], s["work"], s["out"], workspace=s["ws"])
        return s["out"]
    if kind == "dense":
        qsv.sv_apply_dense(s["amps"], s["circuit"], case["k"], layer_begin=1)
        return s["amps"]
    if kind == "branches":
        qsv.sv_batch_run(s["batch"], s["where"], init_plus=True)
        return {"a": s["a"], "b": s["b"]}
    if kind == "uneven":
        qsv.sv_batch_run(s["batch"], s["where"], init_plus=True, bitstrings=s["bits"], m=case["m"],
                         amp_table=s["table"])
        return {"states": s["states"], "table": s["table"]}
    if kind == "combine":
        qsv.sv_branch_combine(s["a"], s["b"], case["branches"], case["m"], s["sign"], s["out"])
        return s["out"]
    if kind == "combine_full":
        na, nb = halves(case)
        qsv.sv_branch_combine_full(s["a"], s["b"], case["branches"], na, nb, left_mask(case), s["fold"][0],
                                   s["fold"][1], s["out"])
        return s["out"]
    if case["op"] == "inner":
        qsv.sv_inner_product(s["a"], s["b"], case["n"], s["out"])
    else:
        qsv.sv_norm_fp64(s["a"], case["n"], s["out"])
    return s["out"]


# --- the circuit family in plain Python, and complex128 results -------------

CYCLE = ("H00", "H01", "V10", "V11", "H10", "V01", "V00", "H11")
DIAGONAL = ("T", "CZ", "PB", "ZB")


def circuit_gates(rows, cols, n, depth, seed):
    """(kind, q0, q1, layer): layer 0 H on all, then the CZ cycle and the
    SplitMix64 draws of T, SX, SY."""
    out = [("H", q, -1, 0) for q in range(n)]
    x, mask = seed & (2 ** 64 - 1), 2 ** 64 - 1
    prev = set()
    for t in range(1, depth + 1):
        way, a, b = CYCLE[(t - 1) % 8]
        a, b = int(a), int(b)
        pairs = []
        for r in range(rows):
            for c in range(cols):
                if way == "H" and c % 2 == a and r % 2 == b and c + 1 < cols:
                    pairs.append((r * cols + c, r * cols + c + 1))
                if way == "V" and r % 2 == a and c % 2 == b and r + 1 < rows:
                    pairs.append((r * cols + c, (r + 1) * cols + c))
        pairs = sorted(p for p in pairs if p[1] < n)
        out += [("CZ", p, q, t) for p, q in pairs]
        now = {q for p in pairs for q in p}
        for q in range(n):
            if q in prev and q not in now:
                x = (x + 0x9E3779B97F4A7C15) & mask
                z = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & mask
                z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
                z ^= z >> 31
                out.append((("T", "SX", "SY")[((z >> 32) * 3) >> 32], q, -1, t))
        prev = now
    return out


def evolve(psi, n, gates, ids=None):
    """The gates on psi (complex128[B, 2^n]), in place; ids: branch index of each row."""
    h = math.sqrt(0.5)
    mats = {"H": (h, h, h, -h), "SX": (.5 + .5j, .5 - .5j, .5 - .5j, .5 + .5j),
            "SY": (.5 + .5j, -.5 - .5j, .5 + .5j, .5 + .5j)}
    rows = psi.shape[0]
    for kind, q, q1, _ in gates:
        if kind == "CZ":
            lo, hi = min(q, q1), max(q, q1)
            psi.view(rows, -1, 2, 1 << (hi - lo - 1), 2, 1 << lo)[:, :, 1, :, 1].neg_()
            continue
        v = psi.view(rows, -1, 2, 1 << q)
        if kind == "T":
            v[:, :, 1] *= complex(h, h)
        elif kind in ("PB", "ZB"):
            bit = ((ids >> q1) & 1).view(rows, 1, 1).to(torch.float64)
            if kind == "PB":
                v[:, :, 0] *= 1 - bit
                v[:, :, 1] *= bit
            else:
                v[:, :, 1] *= 1 - 2 * bit
        else:
            m = mats[kind]
            x = v[:, :, 0].clone()
            v[:, :, 0] *= m[0]
            v[:, :, 0].add_(v[:, :, 1], alpha=m[1])
            v[:, :, 1] *= m[3]
            v[:, :, 1].add_(x, alpha=m[2])
    return psi


def case_gates(case, begin=0):
    n = case["n"]
    return [g for g in circuit_gates(case["rows"], case["cols"], n, case["depth"], case["circuit"]) if g[3] >= begin]


def split_gates(case, seed):
    """Gate lists of both halves: a CZ across the cut is a projector on the
    left and a controlled sign on the right, or only an output sign when no
    non-diagonal gate follows on either qubit."""
    gates = circuit_gates(case["rows"], case["cols"], case["rows"] * case["cols"], case["depth"], seed)
    mask = left_mask(case)
    order = [[q for q in range(case["rows"] * case["cols"]) if (mask >> q) & 1 == side] for side in (1, 0)]
    local = {q: i for side in order for i, q in enumerate(side)}
    last = {}
    for i, g in enumerate(gates):
        if g[0] not in DIAGONAL:
            last[g[1]] = i
    out, cuts = ([], []), 0
    for i, (kind, q, q1, t) in enumerate(gates):
        side = 0 if (mask >> q) & 1 else 1
        if kind == "CZ" and ((mask >> q) & 1) != ((mask >> q1) & 1):
            a, b = (q, q1) if side == 0 else (q1, q)
            if last.get(a, -1) < i and last.get(b, -1) < i:
                continue
            out[0].append(("PB", local[a], cuts, t))
            out[1].append(("ZB", local[b], cuts, t))
            cuts += 1
        else:
            out[side].append((kind, local[q], local[q1] if kind == "CZ" else -1, t))
    return out, cuts


def plus_states(rows, n):
    return torch.full((rows, 1 << n), 2.0 ** (-n / 2), dtype=torch.complex128, device=DEV)


def deposit(positions):
    """Global index of every local index whose bit i is qubit positions[i]."""
    i = torch.arange(1 << len(positions), device=DEV)
    out = torch.zeros_like(i)
    for k, q in enumerate(positions):
        out |= ((i >> k) & 1) << q
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("apply", "dense"):
        n = case["n"]
        psi = random_states(1 << n, 2.0 ** (-n / 2), seed).to(torch.complex128).view(1, -1)
        return evolve(psi, n, case_gates(case, 1)).view(-1)
    if kind == "simulate":
        n = case["n"]
        if case["start"] == "basis":
            psi = torch.zeros(1, 1 << n, dtype=torch.complex128, device=DEV)
            psi[0, random_bits(n, 1, seed + 1)[0]] = 1
            evolve(psi, n, case_gates(case))
        else:
            psi = evolve(plus_states(1, n), n, case_gates(case, 1))
        bits = device_bits(random_bits(n, case["m"], seed))
        return {"state": psi.view(-1), "norm": torch.linalg.vector_norm(psi).square().view(1), "amplitudes": psi[0, bits]}
    if kind == "sample":
        n = case["n"]
        psi = random_states(1 << n, 2.0 ** (-n / 2), seed).to(torch.complex128).view(1, -1)
        return evolve(psi, n, case_gates(case, case["depth"] // 2))[0, device_bits(random_bits(n, case["m"], seed))]
    if kind == "branches":
        gates, cuts = split_gates(case, seed)
        ids = torch.arange(case["branches"], device=DEV) & ((1 << cuts) - 1)
        return {k: evolve(plus_states(case["branches"], n), n, [x for x in g if x[3] > 0], ids)
                for k, n, g in zip("ab", halves(case), gates)}
    if kind == "uneven":
        states, table = [], []
        for i, (n, d, cs) in enumerate(uneven_items(case, seed)):
            rows, cols = lattice(n)
            psi = evolve(plus_states(1, n), n, [g for g in circuit_gates(rows, cols, n, d, cs) if g[3] > 0]).view(-1)
            states.append(psi)
            table.append(psi[device_bits(random_bits(n, case["m"], seed * 64 + i))])
        return {"states": torch.cat(states), "table": torch.cat(table)}
    if kind == "combine":
        s = prepare(case, seed)
        return (s["a"].to(torch.complex128) * s["b"].to(torch.complex128)).sum(0) * s["sign"]
    if kind == "combine_full":
        s = prepare(case, seed)
        na, nb = halves(case)
        mask = left_mask(case)
        ia = deposit([q for q in range(na + nb) if (mask >> q) & 1])
        ib = deposit([q for q in range(na + nb) if not (mask >> q) & 1])
        left, right = folded_pairs(case)
        out = torch.empty(1 << (na + nb), dtype=torch.complex128, device=DEV)
        b = s["b"].to(torch.complex128)
        for rows in torch.arange(1 << na, device=DEV).split(1 << 12):
            part = s["a"][:, rows].to(torch.complex128).t().contiguous() @ b
            odd = torch.zeros(part.shape, dtype=torch.int64, device=DEV)
            for p, q in zip(left, right):
                odd ^= ((ia[rows] >> p) & 1)[:, None] & ((ib >> q) & 1)[None, :]
            out[(ia[rows][:, None] | ib[None, :]).view(-1)] = (part * (1 - 2 * odd)).view(-1)
        return out
    s = prepare(case, seed)
    if case["op"] == "norm":
        return torch.view_as_real(s["a"]).double().square().sum().view(1)
    a, b = (torch.view_as_real(x).double() for x in (s["a"], s["b"]))
    re = (a * b).sum()
    return torch.stack([re, (a[:, 0] * b[:, 1]).sum() - (a[:, 1] * b[:, 0]).sum()])


def work(case):
    """Bytes read and written once; flops = 2 per amplitude and non-diagonal
    gate of a sweep (sum and difference), 8 per complex multiply-add of the
    contractions."""
    kind = case["kind"]
    if kind in ("apply", "simulate", "sample", "dense"):
        first = {"apply": 1, "dense": 1, "sample": case["depth"] // 2}.get(kind, 0 if case.get("start") == "basis" else 1)
        dim = float(1 << case["n"])
        flops = 2.0 * dim * sum(1 for g in case_gates(case, first) if g[0] not in DIAGONAL)
        per = {"apply": 16, "dense": 16, "simulate": 8, "sample": 8}[kind]
        return {"bytes": per * dim + 24.0 * case.get("m", 0), "flops": flops}
    if kind == "branches":
        gates, _ = split_gates(case, 1)
        sizes = [float(case["branches"] << n) for n in halves(case)]
        return {"bytes": 8.0 * sum(sizes),
                "flops": sum(2.0 * d * sum(1 for x in g if x[3] > 0 and x[0] not in DIAGONAL) for d, g in zip(sizes, gates))}
    if kind == "uneven":
        total = flops = 0.0
        for n, d, cs in uneven_items(case, 1):
            rows, cols = lattice(n)
            total += float(1 << n)
            flops += 2.0 * (1 << n) * sum(1 for g in circuit_gates(rows, cols, n, d, cs) if g[3] > 0 and g[0] not in DIAGONAL)
        return {"bytes": 8.0 * total + 24.0 * case["count"] * case["m"], "flops": flops}
    if kind == "combine":
        pairs = float(case["branches"] * case["m"])
        return {"bytes": 16.0 * pairs + 17.0 * case["m"], "flops": 8.0 * pairs}
    if kind == "combine_full":
        na, nb = halves(case)
        return {"bytes": 8.0 * case["branches"] * ((1 << na) + (1 << nb)) + 8.0 * (1 << (na + nb)),
                "flops": 8.0 * case["branches"] * (1 << (na + nb))}
    dim = float(1 << case["n"])
    return {"bytes": dim * (16 if case["op"] == "inner" else 8), "flops": dim * (8 if case["op"] == "inner" else 4)}
