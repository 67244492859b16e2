"""The contractions that users of this package run, as cases to be timed.

Two kinds of work:

* ``pair``: one bit-permuted pairwise contraction C[m, n] = sum_k A[m, k] B[k, n]
  on complex64 tensors (``api.contract_pair``, or ``matnc_contract_noalloc`` for
  callers that hold no scratch buffer).  Every step of a contraction tree is
  one of these.  ``layout`` says how the operands' index bits are stored:
  "plan" as a plan lays its tensors out (contracted bits highest in both
  operands, the rows' and columns' bits interleaved in the result), "shuffled"
  in any order, as a caller with tensors of its own may have them.
* ``amps``: one pass of a plan, from an empty stem cache to the amplitudes of
  a bitstring batch and its linear cross-entropy; ``queue``: one pass over
  several plans of uneven size on one workspace.

A plan's amplitudes come back in the plan's own precision: complex64 plans as
float32 pairs, complex-half plans as float16 pairs in units of 2^(-n/2) (the
size of a random circuit's amplitudes).  The float64 buffer they are taken from
only adds up slices.  The cross-entropy comes back as the mean of x = 2^n |a|^2.

Circuits, bitstrings and operands are made from the seed; contraction trees
belong to the circuit's layout, which does not depend on the seed.
"""

import functools
import json
import math
import os
import shutil
import tempfile

import numpy as np
import torch

import paper_2212_04749_amd
from paper_2212_04749_amd import api, binding, planner
from paper_2212_04749_amd.circuit_tn import build_network

PACKAGE = os.path.dirname(os.path.abspath(paper_2212_04749_amd.__file__))
BUDGET = 56 << 30  # workspace bytes a plan may take

# the uneven batch's circuits whose stored plans take at most a few tenths of
# a second: entry -> (rows, columns, depth, bitstrings, complex MACs)
UNEVEN = {
    2: (5, 5, 12, 4096, 1.72e10), 3: (4, 5, 11, 512, 2.94e8), 4: (5, 5, 12, 256, 1.97e10),
    5: (4, 5, 10, 256, 1.74e8), 6: (4, 6, 16, 256, 1.70e10), 7: (5, 5, 15, 512, 4.09e10),
    8: (4, 7, 13, 512, 9.76e10), 12: (5, 5, 14, 2048, 2.54e10), 13: (4, 5, 16, 1024, 7.37e8),
    21: (4, 5, 10, 1024, 1.38e8), 23: (4, 6, 13, 512, 1.44e10), 25: (4, 7, 10, 256, 5.75e9),
    29: (4, 7, 11, 2048, 1.07e11),
}


def listed():
    return [
        # the smallest step there is: a small tensor times a gate, latency alone
        {"name": "pair_gate_small", "kind": "pair", "nm": 5, "nn": 3, "nk": 2, "batch": 7, "layout": "shuffled",
         "layout_seed": 1, "entry": "scratch"},
        # a small step of a serving loop that allocates nothing
        {"name": "pair_small_noalloc", "kind": "pair", "nm": 12, "nn": 3, "nk": 4, "batch": 3, "layout": "shuffled",
         "layout_seed": 2, "entry": "noalloc"},
        # a two-qubit gate into a large tensor: as many bytes in as out
        {"name": "pair_gate_large", "kind": "pair", "nm": 22, "nn": 2, "nk": 2, "batch": 1, "layout": "plan",
         "layout_seed": 3, "entry": "scratch"},
        # a branch step of the reuse tree: a long sum into a few columns, one per bitstring group
        {"name": "pair_long_sum", "kind": "pair", "nm": 10, "nn": 1, "nk": 11, "batch": 33, "layout": "plan",
         "layout_seed": 4, "entry": "scratch"},
        # columns outnumber rows (the caller passes the small tensor first)
        {"name": "pair_few_rows", "kind": "pair", "nm": 4, "nn": 12, "nk": 5, "batch": 9, "layout": "shuffled",
         "layout_seed": 5, "entry": "scratch"},
        # a middling product of two tensors in an order of the caller's own
        {"name": "pair_gemm", "kind": "pair", "nm": 11, "nn": 7, "nk": 6, "batch": 5, "layout": "shuffled",
         "layout_seed": 6, "entry": "scratch"},
        # the 6x6 circuit's heaviest stem step
        {"name": "pair_stem", "kind": "pair", "nm": 20, "nn": 8, "nk": 9, "batch": 1, "layout": "plan",
         "layout_seed": 7, "entry": "scratch"},
        # the smallest whole job: a 12-qubit circuit in slices, launches alone
        {"name": "amps_3x4_sliced", "kind": "amps", "rows": 3, "cols": 4, "depth": 8, "k": 50, "n_open": 0, "cap": 7,
         "plan": "search", "precision": "c64", "slice_batch": 2, "begin": 0, "end": -1},
        # the fidelity estimate's 20-qubit circuit and its 4096 samples
        {"name": "amps_4x5_fidelity", "kind": "amps", "rows": 4, "cols": 5, "depth": 12, "k": 4096, "n_open": 0,
         "cap": 0, "plan": "search", "precision": "c64", "slice_batch": 1, "begin": 0, "end": -1},
        # 30 qubits, 4096 bitstrings, the stored plan, complex64
        {"name": "amps_5x6", "kind": "amps", "rows": 5, "cols": 6, "depth": 12, "k": 4096, "n_open": 0, "cap": 28,
         "plan": "c2_cap28", "precision": "c64", "slice_batch": 4, "begin": 0, "end": -1},
        # 36 qubits, 64 groups of 2^8 amplitudes, one batch of 8 of the stored plan's 256 slices, complex-half
        {"name": "amps_6x6_slices", "kind": "amps", "rows": 6, "cols": 6, "depth": 14, "k": 64, "n_open": 8,
         "cap": 30, "plan": "c3_cap30", "precision": "chalf", "slice_batch": 8, "begin": 16, "end": 24},
        # six circuits of the uneven batch as one queue, complex-half
        {"name": "queue_uneven", "kind": "queue", "entries": "2,3,5,6,13,21", "precision": "chalf"},
    ]


def draw(rng):
    kind = rng.choices(["gate", "sum", "gemm", "rows", "small", "uneven", "queue"], [3, 2, 4, 2, 3, 3, 1])[0]
    seed = rng.randrange(1 << 20)
    if kind in ("gate", "sum", "gemm", "rows"):
        while True:
            if kind == "gate":  # gates into tensors of every size
                nm, nn, nk = rng.randint(1, 23), rng.randint(0, 4), rng.randint(0, 4)
            elif kind == "sum":
                nm, nn, nk = rng.randint(0, 14), rng.randint(0, 3), rng.randint(5, 13)
            elif kind == "gemm":
                nm, nn, nk = rng.randint(6, 20), rng.randint(5, 9), rng.randint(3, 10)
            else:
                nm, nn, nk = rng.randint(0, 5), rng.randint(5, 14), rng.randint(1, 8)
            batch = int(2 ** rng.uniform(0, 9))
            size = batch * (2 ** (nm + nk) + 2 ** (nn + nk) + 2 ** (nm + nn))
            if size <= 1 << 28 and batch * 2 ** (nm + nn + nk) <= 1 << 36:
                break
        return {"kind": "pair", "nm": nm, "nn": nn, "nk": nk, "batch": batch, "layout": rng.choice(["plan", "shuffled"]),
                "layout_seed": seed, "entry": rng.choice(["scratch", "scratch", "noalloc"])}
    precision = rng.choice(["c64", "chalf"])
    if kind == "small":
        rows, cols = rng.choice([(2, 4), (3, 3), (3, 4), (2, 6), (4, 4)])
        n = rows * cols
        return {"kind": "amps", "rows": rows, "cols": cols, "depth": rng.randint(6, 10),
                "k": max(1, min(2 ** n, int(2 ** rng.uniform(3, 11)))), "n_open": rng.choice([0, 0, 0, 1, 2, 3]),
                "cap": rng.choice([0, n - 4, n - 3]), "plan": "search", "precision": precision,
                "slice_batch": rng.choice([1, 2, 3, 4]), "begin": 0, "end": -1}
    if kind == "uneven":
        i = rng.choice(sorted(UNEVEN))
        rows, cols, depth = UNEVEN[i][:3]
        return {"kind": "amps", "rows": rows, "cols": cols, "depth": depth, "k": int(2 ** rng.uniform(6, 12)),
                "n_open": 0, "cap": 30, "plan": "C5.%d" % i, "precision": precision, "slice_batch": 1, "begin": 0,
                "end": -1}
    some = rng.sample([i for i in sorted(UNEVEN) if UNEVEN[i][4] < 2e10], rng.randint(2, 6))
    return {"kind": "queue", "entries": ",".join(map(str, sorted(some))), "precision": precision}


# ---------------------------------------------------------------------------
# inputs

def circuit(rows, cols, depth, seed):
    """A seeded random grid circuit: depth cycles of a layer of single-qubit
    gates (no repeat on a qubit) and one of fSim gates on the couplers of the
    cycle's pattern, and a last single-qubit layer."""
    rng = np.random.default_rng(seed)
    names, n = ("sqrtX", "sqrtY", "sqrtW"), rows * cols
    last = [None] * n
    layers = []
    for t in range(depth + 1):
        for q in range(n):
            free = [g for g in names if g != last[q]]
            last[q] = free[int(rng.integers(0, len(free)))]
        layers.append({"kind": "1q", "gates": [[q, last[q]] for q in range(n)]})
        if t == depth:
            break
        letter = "ABCDCDAB"[t % 8]
        edges = []
        for r in range(rows):
            for c in range(cols):
                r2, c2 = (r, c + 1) if letter in "AB" else (r + 1, c)
                if (r + c) % 2 == (0 if letter in "AC" else 1) and r2 < rows and c2 < cols:
                    edges.append([r * cols + c, r2 * cols + c2, math.pi / 2, math.pi / 6])
        layers.append({"kind": "2q", "pattern": letter, "gates": sorted(edges)})
    return {"format": "grid-rqc-v1", "kind": "random", "rows": rows, "cols": cols, "removed": [], "n_qubits": n,
            "depth": depth, "seed": seed, "layers": layers}


def bitstrings(n, k, n_open, seed):
    rng = np.random.default_rng(seed + 1000)
    words = rng.integers(0, 1 << n, size=k, dtype=np.uint64)
    return words & np.uint64((1 << (n - n_open)) - 1)  # the highest n_open qubits stay open


@functools.lru_cache(maxsize=None)
def stored(name):
    path = "c5_cap30" if name.startswith("C5.") else name
    with open(os.path.join(PACKAGE, "plans", path + ".json")) as f:
        e = json.load(f)
    e = e[name] if name.startswith("C5.") else e
    return tuple(map(tuple, e["pairs"])), tuple(e["sliced"])


@functools.lru_cache(maxsize=None)
def tree(rows, cols, depth, k, n_open, cap, plan):
    """The contraction tree and sliced indices of a circuit layout, with its cost per pass."""
    net = build_network(circuit(rows, cols, depth, 1))
    words = bitstrings(rows * cols, k, n_open, 1)
    opens = tuple(range(rows * cols - n_open, rows * cols))
    if plan == "search":
        p = planner.find_plan(net, words, opens, cap or None, seed=0, trials=8, refine_top=0)
    else:
        pairs, sliced = stored(plan)
        p = planner.plan_from(net, words, opens, list(pairs), list(sliced))
    return [tuple(x) for x in p.pairs], list(p.sliced), float(p.costs.total)


def tree_of(case):
    return tree(case["rows"], case["cols"], case["depth"], case["k"], case["n_open"], case["cap"], case["plan"])


def entries_of(case):
    """The circuits of a queue as ``amps`` cases."""
    out = []
    for i in map(int, case["entries"].split(",")):
        rows, cols, depth, k, _ = UNEVEN[i]
        out.append({"kind": "amps", "rows": rows, "cols": cols, "depth": depth, "k": k, "n_open": 0, "cap": 30,
                    "plan": "C5.%d" % i, "precision": case["precision"], "slice_batch": 1, "begin": 0, "end": -1})
    return out


def positions(case):
    """Storage bit of each index bit of the three tensors."""
    rng = np.random.default_rng(case["layout_seed"])
    nm, nn, nk = case["nm"], case["nn"], case["nk"]
    if case["layout"] == "plan":
        a, b = list(range(nm + nk)), list(range(nn + nk))
        at = sorted(rng.permutation(nm + nn)[:nm].tolist())
        c = at + [x for x in range(nm + nn) if x not in at]
    else:
        a, b, c = (rng.permutation(r).tolist() for r in (nm + nk, nn + nk, nm + nn))
    return {"posA_m": a[:nm], "posA_k": a[nm:], "posB_n": b[:nn], "posB_k": b[nn:], "posC_m": c[:nm], "posC_n": c[nm:]}


def operands(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.randn((case["batch"], 2 << r), generator=g, device="cuda", dtype=torch.float32)
            for r in (case["nm"] + case["nk"], case["nn"] + case["nk"])]


def contraction(case, seed, **more):
    pairs, sliced, _ = tree_of(case)
    n = case["rows"] * case["cols"]
    net = build_network(circuit(case["rows"], case["cols"], case["depth"], seed))
    opens = tuple(range(n - case["n_open"], n))
    spec = api.PlanSpec(pairs, sliced, opens, case["cap"] or 32)
    return api.Contraction(net, spec, bitstrings(n, case["k"], case["n_open"], seed), precision=case["precision"],
                           slice_batch=case["slice_batch"], memory_budget=BUDGET, **more)


def tune(run):
    """Tile shapes from a copy of the measured choices that ship with the package."""
    fd, path = tempfile.mkstemp(suffix=".json")
    os.close(fd)
    try:
        shutil.copyfile(os.path.join(PACKAGE, "tuning_mi355x.json"), path)
        run.autotune(reps=3, cache_path=path)
    finally:
        os.remove(path)


def amps_like(run):
    """The buffer that a plan's amplitudes are read into, in its own precision."""
    return torch.empty((run.k, 1 << run.n_open, 2), device="cuda",
                       dtype=torch.float32 if run.precision == "c64" else torch.float16)


def unit(case):
    return 1.0 if case["precision"] == "c64" else 2.0 ** (case["rows"] * case["cols"] / 2)


def prepare(case, seed):
    if case["kind"] == "pair":
        a, b = operands(case, seed)
        c = torch.empty((case["batch"], 2 << (case["nm"] + case["nn"])), device="cuda", dtype=torch.float32)
        return {"kind": "pair", "entry": case["entry"], "pos": positions(case), "batch": case["batch"], "a": a, "b": b,
                "c": c}
    if case["kind"] == "amps":
        run = contraction(case, seed)
        if case["plan"] in ("c2_cap28", "c3_cap30"):
            tune(run)
        return {"kind": "amps", "run": run, "sums": run.new_amplitudes(), "amps": amps_like(run), "unit": unit(case),
                "x": torch.empty(1, device="cuda"), "begin": case["begin"],
                "end": case["end"] if case["end"] >= 0 else run.n_slices}
    stream = torch.cuda.Stream()
    cases = entries_of(case)
    runs = [contraction(c, seed + i, stream=stream, bind=False) for i, c in enumerate(cases)]
    queue = api.Queue(runs, shared=True)
    with torch.cuda.stream(stream):
        sums, f = [r.new_amplitudes() for r in runs], torch.zeros(len(runs), dtype=torch.float64, device="cuda")
    return {"kind": "queue", "queue": queue, "runs": runs, "sums": sums, "f": f, "amps": [amps_like(r) for r in runs],
            "units": [unit(c) for c in cases], "x": torch.empty(len(runs), device="cuda")}


# ---------------------------------------------------------------------------

def run(state):
    if state["kind"] == "pair":
        a, b, c, pos = state["a"], state["b"], state["c"], state["pos"]
        if state["entry"] == "scratch":
            state["scratch"] = api.contract_pair(a, b, c, pos)
        else:
            binding.matnc_contract_noalloc(a.data_ptr(), b.data_ptr(), c.data_ptr(), state["batch"], pos["posA_m"],
                                           pos["posA_k"], pos["posB_k"], pos["posB_n"], pos["posC_m"], pos["posC_n"],
                                           -1, torch.cuda.current_stream().cuda_stream)
        return c
    if state["kind"] == "amps":
        plan, sums = state["run"], state["sums"]
        plan.reset_cache()
        with torch.cuda.stream(plan.stream):
            sums.zero_()
        plan.execute(sums, state["begin"], state["end"])
        f = plan.xeb_dev(sums)
        with torch.cuda.stream(plan.stream):
            torch.mul(sums, state["unit"], out=state["amps"])
            torch.add(f, 1.0, out=state["x"])
        return {"amps": state["amps"], "x": state["x"]}
    queue = state["queue"]
    sums, f = queue.execute(state["sums"], state["f"])
    with torch.cuda.stream(queue.stream):
        for s, u, out in zip(sums, state["units"], state["amps"]):
            torch.mul(s, u, out=out)
        torch.add(f, 1.0, out=state["x"])
    return {"amps": state["amps"], "x": state["x"]}


def work(case):
    if case["kind"] == "pair":
        nm, nn, nk, batch = case["nm"], case["nn"], case["nk"], case["batch"]
        return {"bytes": 8 * batch * (2 ** (nm + nk) + 2 ** (nn + nk) + 2 ** (nm + nn)),
                "flops": 8 * batch * 2 ** (nm + nn + nk)}
    total, out = 0.0, 0
    for c in entries_of(case) if case["kind"] == "queue" else [case]:
        _, sliced, cost = tree_of(c)
        part = (c["end"] - c["begin"]) / 2 ** len(sliced) if c["end"] >= 0 else 1.0
        leaves = len(build_network(circuit(c["rows"], c["cols"], c["depth"], 1)).tensors)
        total += 8 * cost * part
        out += (c["k"] << c["n_open"]) * 16 + leaves * 16 * 8
    return {"bytes": out, "flops": total}


# ---------------------------------------------------------------------------
# the same values in 64 bits

S = math.sqrt(0.5)
GATES = {"sqrtX": [[S, -1j * S], [-1j * S, S]], "sqrtY": [[S, -S], [S, S]],
         "sqrtW": [[S, -S * S * (1 + 1j)], [S * S * (1 - 1j), S]]}


def final_state(circ):
    """The circuit's 2^n amplitudes, bit q of the index the value of qubit q."""
    n = circ["n_qubits"]
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1.0
    for layer in circ["layers"]:
        if layer["kind"] == "1q":
            names = dict(layer["gates"])
            for lo in range(0, n, 5):  # gates of five neighbouring qubits as one matrix
                m = np.ones((1, 1))
                for q in range(lo, min(n, lo + 5)):
                    m = np.kron(np.array(GATES[names[q]]), m)
                m = torch.tensor(m, dtype=torch.complex128, device="cuda")
                v = psi.view(-1, m.shape[0], 1 << lo)
                psi = (v[:, :, 0] @ m.t().contiguous() if lo == 0 else torch.matmul(m, v)).reshape(-1)
        else:
            for qa, qb, theta, phi in layer["gates"]:
                lo, hi = min(qa, qb), max(qa, qb)
                v = psi.view(1 << (n - 1 - hi), 2, 1 << (hi - lo - 1), 2, 1 << lo)
                x, y = v[:, 0, :, 1].clone(), v[:, 1, :, 0].clone()
                v[:, 0, :, 1] = math.cos(theta) * x - 1j * math.sin(theta) * y
                v[:, 1, :, 0] = math.cos(theta) * y - 1j * math.sin(theta) * x
                v[:, 1, :, 1] *= complex(math.cos(phi), -math.sin(phi))
    return psi


def exact_amps(case, seed):
    n = case["rows"] * case["cols"]
    psi = final_state(circuit(case["rows"], case["cols"], case["depth"], seed))
    words = torch.from_numpy(bitstrings(n, case["k"], case["n_open"], seed).astype(np.int64)).cuda()
    opened = torch.arange(1 << case["n_open"], device="cuda") << (n - case["n_open"])
    a = psi[words[:, None] + opened[None, :]]
    x = 2.0 ** n * (a.abs() ** 2).mean()
    return torch.view_as_real(a) * unit(case), x


def offsets(pos):
    x = torch.arange(1 << len(pos), device="cuda")
    off = torch.zeros_like(x)
    for t, p in enumerate(pos):
        off |= ((x >> t) & 1) << p
    return off


def exact(case, seed):
    if case["kind"] == "pair":
        a, b = (torch.view_as_complex(t.view(case["batch"], -1, 2)) for t in operands(case, seed))
        at = {k: offsets(p) for k, p in positions(case).items()}
        out = torch.empty((case["batch"], 1 << (case["nm"] + case["nn"])), dtype=torch.complex128, device="cuda")
        rows = max(1, min(1 << case["nm"], (1 << 26) >> case["nk"], (1 << 26) >> case["nn"]))
        for i in range(case["batch"]):
            bm = b[i][at["posB_k"][:, None] + at["posB_n"][None, :]].to(torch.complex128)
            for lo in range(0, 1 << case["nm"], rows):
                am = a[i][at["posA_m"][lo:lo + rows, None] + at["posA_k"][None, :]].to(torch.complex128)
                out[i][at["posC_m"][lo:lo + rows, None] + at["posC_n"][None, :]] = am @ bm
        return torch.view_as_real(out).reshape(case["batch"], -1)
    if case["kind"] == "amps":
        if case["rows"] * case["cols"] > 30:
            return None  # a state vector of 36 qubits does not fit
        a, x = exact_amps(case, seed)
        return {"amps": a, "x": x.reshape(1)}
    each = [exact_amps(c, seed + i) for i, c in enumerate(entries_of(case))]
    return {"amps": [a for a, _ in each], "x": torch.stack([x for _, x in each])}
