"""The work that programs using this framework have it do, as cases that can be timed.

A case is a dict of plain values; its "kind" names the entry point:

  row       Plan.amplitudes, row scheme: amplitudes of one circuit
  square    Plan.amplitudes, square partition
  group     Group.amplitudes: many small circuits in one call
  observe   all <Z_q> and nearest-neighbour <Z_a Z_b> of a state, through its
            double-layer network (network, plan and values in one pass)
  sample    sequential measurement of every qubit
  site      contract_site: one site contraction on the caller's tensors

A case with "shared" has the bitstrings of one base string with the given
number of free qubits at the end of the last row, the others have independent
random bitstrings.  Amplitudes are complex numbers of the plan's precision: a
plan that contracts in FP32 (or BF16x3) gives single-precision mantissas, and a
program keeps them as complex64; an FP64 plan's are kept as complex128.

Needs a GPU for prepare() and run(); work() and listed() do not.
"""
import itertools
import math

import numpy as np
import torch

import paper_1905_08394_amd as psim
import rqcgen

MEM_BUDGET = 32 << 30  # device bytes a plan may use for its workspace
SMALL_LATTICES = ((2, 3), (3, 3), (3, 4), (4, 4), (2, 7), (3, 5), (4, 5), (5, 3))


def listed():
    return [
        # the smallest call: a whole output distribution of nine qubits, replayed as a graph
        {"name": "3x3 all 512", "kind": "row", "lv": 3, "lh": 3, "depth": 8, "bits": 512, "prec": "fp32",
         "split": False, "graph": True},
        # a verification batch of one 20-qubit circuit in the default form of the benchmark
        {"name": "4x5 d24 64", "kind": "row", "lv": 4, "lh": 5, "depth": 24, "bits": 64, "prec": "fp32_3m",
         "split": True, "graph": False},
        # 36 qubits at moderate depth, in the library's default precision
        {"name": "6x6 d24 64", "kind": "row", "lv": 6, "lh": 6, "depth": 24, "bits": 64, "prec": "fp32",
         "split": False, "graph": False},
        # the 25-qubit throughput batch of the parity suite, in the three precisions a user picks from
        {"name": "5x5 d32 256 3M", "kind": "row", "lv": 5, "lh": 5, "depth": 32, "bits": 256, "prec": "fp32_3m",
         "split": True, "graph": False},
        {"name": "5x5 d32 64 FP64", "kind": "row", "lv": 5, "lh": 5, "depth": 32, "bits": 64, "prec": "fp64",
         "split": False, "graph": False},
        {"name": "5x5 d32 256 BF16x3", "kind": "row", "lv": 5, "lh": 5, "depth": 32, "bits": 256, "prec": "bf16x3",
         "split": False, "graph": False},
        # the bond dimension and the bitstring pattern of the 6x6 (1+40+1) benchmark on a lattice of 25 qubits
        {"name": "5x5 d40 16 shared", "kind": "row", "lv": 5, "lh": 5, "depth": 40, "bits": 16, "shared": 4,
         "prec": "fp32_3m", "split": True, "graph": False},
        # random amplitudes of 64 qubits (the statistics workload), through the square partition
        {"name": "8x8 d25 32 square", "kind": "square", "lv": 8, "lh": 8, "depth": 25, "bits": 32, "prec": "fp32_3m",
         "split": False},
        # many small circuits at once, replayed as a graph
        {"name": "48 small circuits", "kind": "group", "count": 48, "bits": 16, "prec": "fp32_3m", "graph": True},
        # every Z and ZZ expectation value of a 20-qubit state
        {"name": "4x5 d16 observables", "kind": "observe", "lv": 4, "lh": 5, "depth": 16, "prec": "fp64", "sweep": 3},
        # measurement shots of a 16-qubit state
        {"name": "4x4 d12 256 shots", "kind": "sample", "lv": 4, "lh": 4, "depth": 12, "samples": 256, "prec": "fp64",
         "sweep": 0},
        # one contraction step on the caller's own tensors, with no size a multiple of a tile
        {"name": "ragged site", "kind": "site", "batch": 6, "M": 20011, "K1": 9, "K2": 6, "N": 75, "prec": "fp32",
         "split": False},
    ]


def draw(rng):
    top = max(_cost(c) for c in listed())

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["row", "row", "row", "row", "square", "square", "group", "observe", "sample", "site"])
        prec = rng.choice(["fp64", "fp32", "fp32_3m", "fp32_3m"] + (["bf16x3"] if kind in ("row", "site") else []))
        split = prec in ("fp32", "fp32_3m") and rng.random() < 0.5
        if kind == "row":
            lv, lh = sorted((rng.randint(2, 6), rng.randint(2, 7)))
            if rng.random() < 0.5:
                lv, lh = lh, lv
            c = {"kind": kind, "lv": lv, "lh": lh, "depth": rng.randint(5, 40), "bits": log_int(1, 400), "prec": prec,
                 "split": split, "graph": rng.random() < 0.3}
            if rng.random() < 0.3:
                c["shared"] = rng.randint(1, min(4, lh))
                c["bits"] = 2 ** c["shared"]
        elif kind == "square":
            c = {"kind": kind, "lv": rng.randint(3, 8), "lh": rng.randint(3, 8), "depth": rng.randint(8, 32),
                 "bits": log_int(1, 200), "prec": prec, "split": split}
        elif kind == "group":
            c = {"kind": kind, "count": log_int(2, 64), "bits": log_int(1, 64), "prec": prec,
                 "graph": rng.random() < 0.5}
        elif kind == "observe":
            c = {"kind": kind, "lv": rng.randint(2, 4), "lh": rng.randint(2, 5), "depth": rng.randint(4, 16),
                 "prec": prec, "sweep": rng.choice([0, 3])}
        elif kind == "sample":
            c = {"kind": kind, "lv": rng.randint(2, 4), "lh": rng.randint(2, 4), "depth": rng.randint(4, 13),
                 "samples": log_int(4, 300), "prec": "fp64", "sweep": rng.choice([0, 3])}
        else:
            c = {"kind": kind, "batch": log_int(1, 16), "M": log_int(64, 60000), "K1": log_int(1, 32),
                 "K2": log_int(1, 32), "N": log_int(1, 512), "prec": prec, "split": split}
        if _cost(c) <= top and _largest(c) <= 2 ** 31:
            return c


# ---------------------------------------------------------------- inputs
def _circuit(case, seed, k=0):
    return rqcgen.generate(case["lv"], case["lh"], case["depth"], 1000 * (seed % 1000003) + k)


def _bits(case, seed):
    lv, lh, n = case["lv"], case["lh"], case["lv"] * case["lh"]
    if case.get("shared"):
        base = rqcgen.bitstrings(lv, lh, seed, 1)[0]
        return rqcgen.last_row_variants(base, lv, lh, list(range(lh - case["shared"], lh)))
    if case["bits"] >= 2 ** n:  # the whole distribution
        return rqcgen.all_bitstrings(n)
    return rqcgen.bitstrings(lv, lh, seed, case["bits"])


def _small(case):
    """The circuits of a group: lattices in turn, depths 8 to 24."""
    return [{"lv": SMALL_LATTICES[k % 8][0], "lh": SMALL_LATTICES[k % 8][1], "depth": 8 + (5 * k) % 17,
             "bits": case["bits"]} for k in range(case["count"])]


def _observable_bits(case):
    """With the slices (Z, I) at every site: 0 where a product has a Z, 1 elsewhere."""
    lv, lh = case["lv"], case["lh"]
    n = lv * lh
    sets = [()] + [(q,) for q in range(n)] + list(rqcgen.lattice_edges(lv, lh))
    b = np.ones((len(sets), n), dtype=np.uint8)
    for row, qs in zip(b, sets):
        row[list(qs)] = 0
    return b, sets


def _site_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.complex128 if case["prec"] == "fp64" else torch.complex64
    A = torch.randn(case["batch"] * case["K1"] * case["M"] * case["K2"], dtype=dt, device="cuda", generator=g)
    r = np.random.default_rng(seed)
    W = r.standard_normal((case["K1"] * case["K2"], case["N"], 2)).astype(np.float32).astype(np.float64)
    return A, W.view(np.complex128)[..., 0]


def _plan(circuit, n, **kw):
    peps = psim.Peps(circuit)
    plan = psim.Plan(peps, max_batch=n, mem_budget=MEM_BUDGET, **kw)
    peps.close()
    plan.workspace()
    return plan


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("row", "square"):
        bits = _bits(case, seed)
        plan = _plan(_circuit(case, seed), len(bits), prec=case["prec"], split_acc=case["split"],
                     sweep=3 if kind == "square" else 0, graph=case.get("graph", False))
        return {"case": case, "plan": plan, "bits": bits}
    if kind == "group":
        cs = _small(case)
        bits = [_bits(c, seed + k) for k, c in enumerate(cs)]
        plans = [_plan(_circuit(c, seed, k), len(b), prec=case["prec"], graph=case["graph"])
                 for k, (c, b) in enumerate(zip(cs, bits))]
        return {"case": case, "plans": plans, "group": psim.Group(plans), "bits": bits}
    if kind == "observe":
        return {"case": case, "peps": psim.Peps(_circuit(case, seed)), "bits": _observable_bits(case)[0]}
    if kind == "sample":
        u = np.random.default_rng(seed).random((case["samples"], case["lv"] * case["lh"]))
        return {"case": case, "peps": psim.Peps(_circuit(case, seed)), "u": u}
    A, W = _site_inputs(case, seed)
    return {"case": case, "A": A, "W": W}


def run(state):
    case = state["case"]
    kind, prec = case["kind"], case["prec"]
    if kind in ("row", "square"):
        return _keep(state["plan"].amplitudes(state["bits"]), prec)
    if kind == "group":
        return _keep(np.concatenate(state["group"].amplitudes(state["bits"])), prec)
    if kind == "observe":
        n = case["lv"] * case["lh"]
        ops = np.zeros((n, 2, 2, 2), dtype=complex)
        ops[:, 0] = np.diag([1.0, -1.0])
        ops[:, 1] = np.eye(2)
        network = state["peps"].double_layer(ops)
        plan = psim.Plan(network, prec=prec, max_batch=len(state["bits"]), sweep=case["sweep"], mem_budget=MEM_BUDGET)
        values = plan.amplitudes(state["bits"])
        plan.close()
        network.close()
        return _keep(values, prec)
    if kind == "sample":
        return psim.sample(state["peps"], state["u"], prec=prec, sweep=case["sweep"],
                           max_batch=2 * case["samples"], mem_budget=MEM_BUDGET)
    return psim.contract_site(prec, state["A"], state["W"], case["M"], case["K1"], case["K2"], case["N"],
                              batch=case["batch"], split_acc=case["split"])


def _keep(amps, prec):
    return amps if prec == "fp64" else amps.astype(np.complex64)


# ---------------------------------------------------------------- counts
def _legs(case):
    """Bond sizes of the network: {(site, site): size}, every CZ doubling its bond (squared for a double layer)."""
    bond = {}
    for t in range(case["depth"]):
        for e in rqcgen.coupler_pattern(case["lv"], case["lh"], t % 8):
            bond[e] = bond.get(e, 1) * 2
    if case["kind"] in ("observe", "sample"):
        bond = {e: b * b for e, b in bond.items()}
    return bond


def _row_rows(case):
    """Complex multiply-adds of each row of the row scheme, for one bitstring, and its largest tensor."""
    bond, lv, lh = _legs(case), case["lv"], case["lh"]
    rows, cols = (lv, lh) if lh <= lv else (lh, lv)

    def size(a, b):  # bond between sweep sites (row, column) a and b, 1 outside the lattice
        if not all(0 <= x[0] < rows and 0 <= x[1] < cols for x in (a, b)):
            return 1
        q = [x[0] * lh + x[1] if lh <= lv else x[1] * lh + x[0] for x in (a, b)]
        return bond.get((q[0], q[1]), 1)

    out, largest = [], 1
    for i in range(rows):
        total = 0
        up = [size((i - 1, j), (i, j)) for j in range(cols)]
        down = [size((i, j), (i + 1, j)) for j in range(cols)]
        for j in range(cols):
            l, r = size((i, j - 1), (i, j)), size((i, j), (i, j + 1))
            m = math.prod(up[j + 1:]) * math.prod(down[:j])
            total += m * up[j] * l * down[j] * r
            largest = max(largest, m * down[j] * r)
        out.append(total)
    return out, largest


def _square_parts(case):
    """Complex multiply-adds of the four quadrants (each with its number of sites) and the two joins of the square
    partition, and its largest quadrant tensor."""
    bond, lv, lh = _legs(case), case["lv"], case["lh"]
    a, b = lv // 2, lh // 2

    def size(p, q):
        p, q = sorted((p, q))
        if p[0] < 0 or p[1] < 0 or q[0] >= lv or q[1] >= lh:
            return 1
        return bond.get((p[0] * lh + p[1], q[0] * lh + q[1]), 1)

    quads, open_legs = [], []
    for low, right in ((0, 0), (0, 1), (1, 0), (1, 1)):
        rs = list(range(a)) if not low else list(range(lv - 1, a - 1, -1))
        cs = list(range(b)) if not right else list(range(lh - 1, b - 1, -1))
        dr, dc = (-1 if low else 1), (-1 if right else 1)
        total, side, up = 0, 1, [1] * len(cs)
        for i in rs:
            left, down = 1, []
            for k, j in enumerate(cs):
                d, r = size((i, j), (i + dr, j)), size((i, j), (i, j + dc))
                total += math.prod(up[k + 1:]) * side * math.prod(down) * up[k] * left * d * r
                down.append(d)
                left = r
            side *= left
            up = down
        quads.append((total, len(rs) * len(cs)))
        open_legs.append((math.prod(up), side))  # (vertical cut, horizontal cut)
    (v_ul, h_u), (v_ur, _), (_, h_l), _ = open_legs
    return quads, [v_ur * h_u * v_ul, v_ur * v_ul * h_l], max(v * h for v, h in open_legs)


def _bitstring_count(case):
    n = case["lv"] * case["lh"]
    return min(case["bits"], 2 ** n)


def _cmac(case):
    kind = case["kind"]
    if kind == "group":
        return sum(_cmac({**c, "kind": "row"}) for c in _small(case))
    if kind == "site":
        return case["batch"] * case["M"] * case["K1"] * case["K2"] * case["N"]
    if kind == "row":
        rows, _ = _row_rows(case)
        n, width = _bitstring_count(case), min(case["lv"], case["lh"])
        if case.get("shared"):  # one contraction of all rows but the last
            return sum(rows[:-1]) + n * rows[-1]
        return sum(min(n, 2 ** (width * (i + 1))) * r for i, r in enumerate(rows))
    if kind == "observe":
        n = 1
    elif kind == "sample":  # one network per qubit, both of its values for every prefix: at least one contraction each
        n = case["lv"] * case["lh"]
    else:
        n = _bitstring_count(case)
    if kind == "square" or case["sweep"] == 3:
        quads, joins, _ = _square_parts(case)
        return n * sum(joins) + sum(min(n, 2 ** sites) * total for total, sites in quads)
    return n * sum(_row_rows(case)[0])


def _largest(case):
    """Elements of the largest tensor the pass holds for one bitstring."""
    if case["kind"] == "group":
        return 1
    if case["kind"] == "site":
        return case["batch"] * case["M"] * (case["K1"] * case["K2"] + case["N"])
    if case["kind"] == "square" or case.get("sweep") == 3:
        return 16 * _square_parts(case)[2]
    return _row_rows(case)[1]


def _cost(case):
    """Multiply-adds, weighted by how much longer FP64 takes; used to keep drawn cases below the largest listed one."""
    return _cmac(case) * (3 if case["prec"] == "fp64" else 1)


def work(case):
    flops = 8.0 * _cmac(case)
    e = 16 if case["prec"] == "fp64" else 8
    if case["kind"] == "site":
        b = case["batch"]
        k = case["K1"] * case["K2"]
        return {"bytes": float(e * (b * case["M"] * (k + case["N"])) + 16 * k * case["N"]), "flops": flops}
    if case["kind"] == "group":
        parts = [({**c, "kind": "row", "prec": case["prec"]}) for c in _small(case)]
        return {"bytes": sum(work(p)["bytes"] for p in parts), "flops": flops}
    # every site matrix once (both values of its qubit), the bitstrings, the results
    n = case["lv"] * case["lh"]
    bond = _legs(case)
    site = [1] * n
    for (a, b), size in bond.items():
        site[a] *= size
        site[b] *= size
    count = case["samples"] if case["kind"] == "sample" else \
        len(_observable_bits(case)[0]) if case["kind"] == "observe" else _bitstring_count(case)
    return {"bytes": float(2 * e * sum(site) + count * (n + 16)), "flops": flops}


# ---------------------------------------------------------------- 64-bit values
def _matrices():
    h = math.sqrt(0.5)
    sx = 0.5 * np.array([[1 + 1j, 1 - 1j], [1 - 1j, 1 + 1j]])
    sy = 0.5 * np.array([[1 + 1j, -1 - 1j], [1 + 1j, 1 + 1j]])
    return {k: torch.tensor(np.asarray(v, dtype=complex), device="cuda") for k, v in
            {"H": [[h, h], [h, -h]], "T": [[1, 0], [0, np.exp(0.25j * np.pi)]], "SX": sx, "SY": sy}.items()}


def _state(circuit):
    """State vector, one axis per qubit."""
    n, mats = circuit.n_qubits, _matrices()
    psi = torch.zeros((2,) * n, dtype=torch.complex128, device="cuda")
    psi[(0,) * n] = 1
    for g in circuit.gates:
        if g.kind == "CZ":
            at = [slice(None)] * n
            at[g.q0] = at[g.q1] = 1
            psi[tuple(at)] *= -1
        else:
            psi = torch.movedim(torch.tensordot(mats[g.kind], psi, dims=([1], [g.q0])), 0, g.q0)
    return psi


def _network(circuit):
    """Site tensors [value][left][right][up][down] of the circuit's state; a CZ is sum_s |s><s| x Z^s."""
    mats = {k: v.cpu().numpy() for k, v in _matrices().items()}
    site = [np.array([1, 0], dtype=complex).reshape(2, 1, 1, 1, 1) for _ in range(circuit.n_qubits)]
    one = np.zeros((2, 2, 2))  # [s][value'][value]
    one[0, 0, 0] = one[1, 1, 1] = 1
    two = np.array([np.eye(2), np.diag([1.0, -1.0])])
    for g in circuit.gates:
        if g.kind != "CZ":
            site[g.q0] = np.tensordot(mats[g.kind], site[g.q0], axes=([1], [0]))
            continue
        across = g.q1 == g.q0 + 1
        for q, axis, split in ((g.q0, 2 if across else 4, one), (g.q1, 1 if across else 3, two)):
            t = np.moveaxis(np.tensordot(split, site[q], axes=([2], [0])), 0, axis + 1)  # bond, s
            site[q] = t.reshape(t.shape[:axis] + (t.shape[axis] * 2,) + t.shape[axis + 2:])
    return [torch.tensor(t, device="cuda") for t in site]


def _amplitudes(circuit, bits):
    """Row by row, bitstrings that agree on the rows so far together."""
    lv, lh = circuit.lv, circuit.lh
    site = _network(circuit)
    if lh <= lv:
        grid = [[r * lh + c for c in range(lh)] for r in range(lv)]
        order = (2, 0, 3, 1)  # [left][right][up][down] -> [up][left][down][right]
    else:
        grid = [[r * lh + c for r in range(lv)] for c in range(lh)]
        order = (0, 2, 1, 3)  # the same, rows and columns exchanged
    out = np.zeros(len(bits), dtype=complex)

    def descend(i, F, which):
        if i == len(grid):
            out[which] = complex(F.reshape(-1)[0])
            return
        key = lambda b: tuple(bits[b][grid[i]])  # noqa: E731
        for values, group in itertools.groupby(sorted(which, key=key), key=key):
            T = F.unsqueeze(-1)  # [up ...][down ...][right]
            for q, v in zip(grid[i], values):
                T = torch.tensordot(T, site[q][int(v)].permute(order), dims=([0, T.dim() - 1], [0, 1]))
            descend(i + 1, T.squeeze(-1), list(group))

    descend(0, torch.ones((1,) * len(grid[0]), dtype=torch.complex128, device="cuda"), list(range(len(bits))))
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("row", "square"):
        return _amplitudes(_circuit(case, seed), _bits(case, seed))
    if kind == "group":
        return np.concatenate([_amplitudes(_circuit(c, seed, k), _bits(c, seed + k))
                               for k, c in enumerate(_small(case))])
    if kind == "observe":
        p = _state(_circuit(case, seed)).abs() ** 2
        sets = _observable_bits(case)[1]
        z = torch.tensor([1.0, -1.0], dtype=torch.float64, device="cuda")
        out = []
        for qs in sets:
            v = p
            for q in qs:
                v = v * z.reshape([2 if k == q else 1 for k in range(p.dim())])
            out.append(complex(v.sum().item()))
        return np.array(out)
    if kind == "sample":
        n = case["lv"] * case["lh"]
        u = np.random.default_rng(seed).random((case["samples"], n))
        p = (_state(_circuit(case, seed)).abs() ** 2).cpu().numpy()
        bits, prob = np.zeros(u.shape, dtype=np.uint8), np.zeros(len(u))
        for s, row in enumerate(u):
            left = p
            for k in range(n):
                w = left.reshape(2, -1).sum(axis=1)
                bits[s, k] = 0 if row[k] < w[0] / w.sum() else 1
                left = left[bits[s, k]]
            prob[s] = left
        return bits, prob
    A, W = _site_inputs(case, seed)
    k1, k2 = case["K1"], case["K2"]
    A = A.to(torch.complex128).reshape(case["batch"], k1, case["M"], k2).permute(0, 2, 1, 3)
    return (A.reshape(-1, k1 * k2) @ torch.tensor(np.ascontiguousarray(W), device="cuda")).reshape(-1)
