"""The work that users of this library have it do, as cases that can be timed and compared.

Three kinds of pass, each through the package's public entry points:

circuit   One contraction of a random circuit's network along a planned path, every slice
          summed: `Contraction.contract`.  3 x 4 / 8 cycles (the smallest network) up to the
          30-qubit, 14-cycle one with 1024 slices, in complex64 and both split precisions,
          for one group of many open qubits, for single bitstrings and for many groups.
share     One GPU's share of the 53-qubit, 20-cycle circuit: a subset of the slices of a
          98-bond slicing, 2^14 groups of 64 amplitudes, along the branch-merged path; with
          reuse > 1 the slices come as subtasks whose head is contracted once.
draws     Bitstrings drawn from amplitudes on the GPU: `Contraction.sample`.

The path and the sliced bonds depend on the circuit's structure alone, so they are searched
once per structure and kept, as a program that contracts many circuits of one device does;
gates, angles, targets and slice ids come from the seed.  Every two-qubit gate has an angle of
its own near pi/2, as calibrated gates have.  Amplitudes are contracted in single precision and
summed in double; a pass returns them as complex64, the precision they carry.
"""

import functools
import math

import numpy as np
import torch

from paper_2111_03011_amd import tnc
from paper_2111_03011_amd.contractor import Contraction
from paper_2111_03011_amd.network import circuit_network
from paper_2111_03011_amd.planner import find_plan, merge_branches, order_for_reuse

FORMS = {"c64": tnc.TNC_C64, "bf16x3": tnc.TNC_BF16X3, "fp16x3": tnc.TNC_FP16X3}
SHARE_OPEN = (11, 19, 28, 29, 37, 44)
LARGEST_FLOPS = 4.0e13   # the listed 30-qubit pass


def _circuit_case(name, rows, cols, cycles, n_open, groups, sliced, form, batch, merged=False,
                  norm=False):
    return {"name": name, "kind": "circuit", "rows": rows, "cols": cols, "cycles": cycles,
            "n_open": n_open, "groups": groups, "sliced": sliced, "form": form, "batch": batch,
            "merged": merged, "norm": norm}


def listed():
    return [
        # a few amplitudes of a small circuit: a validation or calibration loop, all latency
        _circuit_case("small_amplitudes", 3, 4, 8, 0, 64, 0, "c64", 1),
        # the whole state of the same small circuit in a split precision
        _circuit_case("small_state_fp16x3", 3, 4, 8, 12, 1, 0, "fp16x3", 1),
        # a served request: correlated amplitudes of a mid-size circuit, batch left to the library
        _circuit_case("request_amplitudes", 4, 6, 12, 6, 64, 6, "c64", 0, merged=True, norm=True),
        # a served request for thousands of uncorrelated samples: one group of 64 for each
        _circuit_case("request_samples", 4, 5, 11, 6, 5000, 4, "c64", 0, merged=True, norm=True),
        # the 30-qubit workload in every form: all 1024 slices of one group of 4096 amplitudes
        _circuit_case("sliced_c64", 5, 6, 14, 12, 1, 10, "c64", 64),
        _circuit_case("sliced_bf16x3", 5, 6, 14, 12, 1, 10, "bf16x3", 64),
        _circuit_case("sliced_fp16x3", 5, 6, 14, 12, 1, 10, "fp16x3", 64),
        # one launch sequence of the 53-qubit share (the large-scale run), and in split precision
        {"name": "share_c64", "kind": "share", "slices": 64, "batch": 64, "reuse": 1, "form": "c64"},
        {"name": "share_bf16x3", "kind": "share", "slices": 64, "batch": 64, "reuse": 1, "form": "bf16x3"},
        # the same circuit as subtasks of 8 slices that share their head
        {"name": "share_reuse_c64", "kind": "share", "slices": 64, "batch": 8, "reuse": 8, "form": "c64"},
        # samples from one group of correlated amplitudes (the 30-qubit workload's)
        {"name": "draws_one_group", "kind": "draws", "n_open": 12, "groups": 1, "samples": 1000},
        # one sample from each of the 53-qubit share's groups
        {"name": "draws_groups", "kind": "draws", "n_open": 6, "groups": 16384, "samples": 16384},
    ]


def draw(rng):
    kind = rng.choice(["circuit", "circuit", "circuit", "share", "draws"])
    form = rng.choice(["c64", "c64", "bf16x3", "fp16x3"])
    if kind == "share":
        reuse = rng.choice([1, 1, 8])
        slices = rng.randint(9, 64) if reuse == 1 else 8 * rng.randint(2, 16)
        return {"kind": "share", "slices": slices, "batch": 8 if reuse == 8 else rng.choice([16, 32, 64]),
                "reuse": reuse, "form": form}
    if kind == "draws":
        if rng.random() < 0.5:
            return {"kind": "draws", "n_open": rng.randint(5, 14), "groups": 1,
                    "samples": int(2 ** rng.uniform(6, 16))}
        groups = int(2 ** rng.uniform(6, 14))
        return {"kind": "draws", "n_open": rng.randint(3, 7), "groups": groups, "samples": groups}
    while True:
        rows, cols = rng.choice([(3, 3), (3, 4), (3, 5), (4, 4), (3, 6), (4, 5), (4, 6), (5, 5), (4, 7)])
        n = rows * cols
        cycles = rng.randint(6, 14)
        n_open = rng.choice([0, 4, 6, 6, 8, 10])
        n_open = min(n_open, n)
        groups = 1 if n_open >= 8 else int(2 ** rng.uniform(0, min(n - n_open - 1, 12)))
        sliced = 0 if n < 16 else rng.randint(0, 8)
        case = {"kind": "circuit", "rows": rows, "cols": cols, "cycles": cycles, "n_open": n_open,
                "groups": groups, "sliced": sliced, "form": form,
                "batch": 0 if sliced else 1, "merged": bool(sliced) and rng.random() < 0.7,
                "norm": rng.random() < 0.5}
        try:
            plan, _ = _plan(*_structure(case))
        except RuntimeError:      # no plan with that many slices fits the size bound
            continue
        if plan.total_flops <= LARGEST_FLOPS:
            return case


# ---- inputs -----------------------------------------------------------------------------------
def _circuit(rows, cols, cycles, seed, jitter, removed=()):
    """A random circuit on a grid: cycles of single-qubit gates that never repeat on a qubit,
    then two-qubit gates on the coupler pattern of the sequence ABCDCDAB; angles
    pi/2 + jitter * normal."""
    sites = [(r, c) for r in range(rows) for c in range(cols) if (r, c) not in removed]
    at = {s: i for i, s in enumerate(sites)}
    rng = np.random.default_rng(seed)
    names = ("sqrt_x", "sqrt_y", "sqrt_w")
    last = rng.integers(0, 3, len(sites))
    layers = []
    for t in range(cycles):
        if t:
            last = (last + rng.integers(1, 3, len(sites))) % 3
        p = "ABCDCDAB"[t % 8]
        step = (0, 1) if p in "AB" else (1, 0)
        pairs = sorted((q, at[(r + step[0], c + step[1])]) for (r, c), q in at.items()
                       if (c if p in "AB" else r) % 2 == "ABCD".index(p) % 2
                       and (r + step[0], c + step[1]) in at)
        layers.append({"oneq": [names[i] for i in last], "couplers": [list(x) for x in pairs]})
    n2 = sum(len(x["couplers"]) for x in layers)
    theta = [float(x) for x in math.pi / 2 + jitter * rng.standard_normal(n2)]
    return {"n_qubits": len(sites), "cycles": cycles, "layers": layers,
            "fsim": {"theta": math.pi / 2, "phi": math.pi / 6, "thetas": theta}}


def _targets(n, open_qubits, groups, seed):
    """Distinct closed parts of the groups: coin flips on the closed qubits."""
    rng = np.random.default_rng([seed, 7])
    closed = [q for q in range(n) if q not in set(open_qubits)]
    if len(closed) <= 20:
        v = rng.choice(1 << len(closed), groups, replace=False).astype(np.uint64)
    else:
        v = np.zeros(0, np.uint64)
        while len(v) < groups:
            v = np.unique(np.concatenate([v, rng.integers(0, 1 << len(closed), 2 * groups, dtype=np.uint64)]))
        v = rng.permutation(v)[:groups]
    out = np.zeros(groups, np.uint64)
    for b, q in enumerate(closed):
        out |= ((v >> np.uint64(b)) & np.uint64(1)) << np.uint64(n - 1 - q)
    return out


def _open(case):
    n = case["rows"] * case["cols"]
    return tuple(range(n - case["n_open"], n))


def _structure(case):
    if case["kind"] == "share":
        return 6, 9, 20, ((0, 4),), SHARE_OPEN, 1 << 14, None, 30.0, True, 1, 5004, case["reuse"]
    return (case["rows"], case["cols"], case["cycles"], (), _open(case), case["groups"],
            case["sliced"], 26.0, case["merged"], 64, 2005, 1)


@functools.lru_cache(maxsize=None)
def _plan(rows, cols, cycles, removed, open_qubits, groups, sliced, max_log2, merged, trials, path_seed, reuse):
    """The path and the sliced bonds of a circuit structure, searched on one circuit of it, and
    how many slices the whole sum has."""
    circ = _circuit(rows, cols, cycles, 1, 0.0, removed)
    net, closed = circuit_network(circ), _targets(circ["n_qubits"], open_qubits, groups, 1)
    plan = find_plan(net, open_qubits, closed, max_log2=max_log2, n_sliced=sliced, trials=trials, seed=path_seed)
    if merged:
        plan = merge_branches(net, plan, open_qubits, closed)
    if reuse > 1:
        plan = order_for_reuse(net, plan, open_qubits, closed, reuse)
    return plan, len(plan.sliced_labels)


def _problem(case, seed):
    """(circuit, open qubits, closed bits, plan, slice ids) of a case."""
    s = _structure(case)
    plan, k = _plan(*s)
    circ = _circuit(s[0], s[1], s[2], seed, 0.02 if case["kind"] == "share" else 0.1, s[3])
    closed = _targets(circ["n_qubits"], s[4], s[5], seed)
    if case["kind"] != "share":
        return circ, s[4], closed, plan, np.arange(1 << k, dtype=np.uint64)
    local = case["reuse"].bit_length() - 1
    rng = np.random.default_rng([seed, 11])
    heads = set()
    while len(heads) < case["slices"] // case["reuse"]:
        heads.add(int.from_bytes(rng.bytes(16), "little") >> (128 - (k - local)))
    ids = [(h << local) | x for h in sorted(heads) for x in range(case["reuse"])]
    return circ, s[4], closed, plan, np.asarray(ids, dtype=object)


def _draws_amps(case, seed):
    """Amplitudes as a random circuit's are: complex normal (their squares exponential)."""
    shape = (case["groups"], 1 << case["n_open"], 2)
    x = np.random.default_rng(seed).standard_normal(shape) * 2.0 ** -15
    return torch.from_numpy(x[..., 0] + 1j * x[..., 1])


def prepare(case, seed):
    if case["kind"] == "draws":
        # a contraction whose groups and open qubits are the case's; its path is the least work
        n = case["n_open"] + max(1, (case["groups"] - 1).bit_length())
        rows = 3
        cols = -(-n // rows)
        n = rows * cols
        circ = _circuit(rows, cols, 4, seed, 0.1)
        open_q = tuple(range(n - case["n_open"], n))
        closed = _targets(n, open_q, case["groups"], seed)
        plan, _ = _plan(rows, cols, 4, (), open_q, case["groups"], 0, 26.0, False, 1, 1, 1)
        c = Contraction(circuit_network(circ), plan.path, open_qubits=open_q, closed_bits=closed)
        c.amps.copy_(_draws_amps(case, seed))
        return {"case": case, "c": c, "seed": seed}
    circ, open_q, closed, plan, ids = _problem(case, seed)
    c = Contraction(circuit_network(circ), plan.path, sliced_labels=plan.sliced_labels, slice_ids=ids,
                    open_qubits=open_q, closed_bits=closed, precision=FORMS[case["form"]],
                    max_batch_slices=case["batch"])
    return {"case": case, "c": c, "seed": seed}


def run(state):
    case, c = state["case"], state["c"]
    if case["kind"] == "draws":
        return {"bits": c.sample(state["seed"], case["samples"]).view(np.int64)}
    if case.get("norm"):
        norm = c.contract(norm=True)
        return {"amps": c.amps.to(torch.complex64), "norm": float(norm)}
    c.contract()
    return {"amps": c.amps.to(torch.complex64)}


def work(case):
    """Circuits: the multiply-adds of the planned path (8 real operations each) and the
    amplitudes written; draws: every amplitude read, every bitstring written."""
    if case["kind"] == "draws":
        n = case["groups"] << case["n_open"]
        return {"bytes": 16.0 * n + 8.0 * case["samples"], "flops": 4.0 * n}
    plan, k = _plan(*_structure(case))
    n_amps = (1 << 20) if case["kind"] == "share" else case["groups"] << case["n_open"]
    slices = case["slices"] if case["kind"] == "share" else 1 << k
    # steps above the bonds that the slices of a subtask share are counted once for each subtask
    return {"bytes": 8.0 * n_amps, "flops": plan.cost.total(slices)}


# ---- what the outputs are, in 64 bits -----------------------------------------------------------
def _state_vector(circ):
    """The circuit's state in complex128, gate by gate, as a flat tensor (qubit 0 is the top bit)."""
    n = circ["n_qubits"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=dev)
    psi[0] = 1.0
    x, y = np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]])
    gate = {k: (np.eye(2) - 1j * p) / math.sqrt(2)
            for k, p in (("sqrt_x", x), ("sqrt_y", y), ("sqrt_w", (x + y) / math.sqrt(2)))}
    thetas = iter(circ["fsim"]["thetas"])
    phase = complex(np.exp(-1j * circ["fsim"]["phi"]))
    for layer in circ["layers"]:
        for q, name in enumerate(layer["oneq"]):
            v, u = psi.view(1 << q, 2, -1), gate[name]
            a, b = v[:, 0], v[:, 1]
            t = a * complex(u[1, 0])
            a.mul_(complex(u[0, 0])).add_(b, alpha=complex(u[0, 1]))
            b.mul_(complex(u[1, 1])).add_(t)
            del t
        for qa, qb in layer["couplers"]:
            th = next(thetas)
            v = psi.view(1 << qa, 2, 1 << (qb - qa - 1), 2, -1)
            a, b = v[:, 0, :, 1], v[:, 1, :, 0]
            t = a * complex(0, -math.sin(th))
            a.mul_(math.cos(th)).add_(b, alpha=complex(0, -math.sin(th)))
            b.mul_(math.cos(th)).add_(t)
            v[:, 1, :, 1].mul_(phase)
            del t
    return psi


def exact(case, seed):
    # the 53-qubit share's slices have no reference that 20 seconds allow; draws are whole numbers
    if case["kind"] != "circuit":
        return None
    circ, open_q, closed, _, _ = _problem(case, seed)
    n, n_open = circ["n_qubits"], len(open_q)
    mu = np.arange(1 << n_open, dtype=np.int64)
    off = np.zeros(1 << n_open, np.int64)
    for t, q in enumerate(open_q):
        off |= ((mu >> (n_open - 1 - t)) & 1) << (n - 1 - q)
    psi = _state_vector(circ)
    at = torch.from_numpy(closed.astype(np.int64)[:, None] + off[None, :]).to(psi.device)
    amps = psi[at]
    out = {"amps": amps}
    if case["norm"]:
        out["norm"] = float((amps.real ** 2 + amps.imag ** 2).sum())
    return out
