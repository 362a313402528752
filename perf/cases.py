"""Performance cases of the sliced state-vector path.

Each case is a piece of work that a program built on this package does through
its public entry points (`paper_1910_09534_amd.sv`, `planner`, `runner`,
`include/sv.h`):

  circuit   one planned ABCDCDAB circuit on a resident state: sv_reset,
            apply_ops, reduce_slices (what the benchmark times, and what the
            server does for each request)
  batch     many circuits recorded as one graph-captured batch and replayed
  sliced    a sliced run: phases with alternating sliced sets, a permute at
            each phase switch, slices resident or in the pinned host tier
  block     one aggregate gate on a dense state (apply_fused, sync_state)
  diag      one diagonal gate on a dense state (apply_diag, sync_state)
  permute   one re-layout of a resident state (permute_qubits)
  contract  the contraction of two tensors over their entanglement indices

`listed()` holds the sizes that stand for them, `draw()` gives more of the same
ranges, `prepare()` makes what a program has in hand before the call, `run()` is
one pass, `work()` what a pass cannot do without and `exact()` its result in 64
bits with plain torch.
"""
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_1910_09534_amd import planner, runner, sv
from paper_1910_09534_amd import workload as W

AMP = {"c64": 8, "c128": 16}
TORCH = {"c64": torch.complex64, "c128": torch.complex128}
NUMPY = {"c64": np.complex64, "c128": np.complex128}
# what a caller keeps of the FP64 sums: the precision of the state they come from
REAL = {"c64": np.float32, "c128": np.float64}
# near-square grids on which the corner and centre slice sets are disjoint in every gate
SLICED_N = (16, 17, 20, 23, 24, 25)


def listed():
    return [
        # the headline: 30 qubits (5 x 6 grid), depth 14, blocks of at most 5 qubits, 2^16 amplitudes
        {"name": "circuit 30q d14 c64", "kind": "circuit", "n": 30, "depth": 14, "dtype": "c64", "kmax": 5,
         "bits": 1 << 16, "plan": "full"},
        # the smallest configuration: 4 x 4 grid, depth 8, every amplitude, in double
        {"name": "circuit 16q d8 c128", "kind": "circuit", "n": 16, "depth": 8, "dtype": "c128", "kmax": 4,
         "bits": 1 << 16, "plan": "full"},
        # the double-precision reference form of a request of ordinary size
        {"name": "circuit 26q d14 c128", "kind": "circuit", "n": 26, "depth": 14, "dtype": "c128", "kmax": 5,
         "bits": 1024, "plan": "fast"},
        # a batch of independent circuits of uneven size, replayed as one graph
        {"name": "batch 16 x 20-24q c64", "kind": "batch", "count": 16, "nmin": 20, "nmax": 24, "dmin": 10,
         "dmax": 20, "bits": 1024},
        # slices staged through the secondary tier, an all-to-all between the phases
        {"name": "sliced 24q d12 tier c64", "kind": "sliced", "n": 24, "depth": 12, "dtype": "c64", "kmax": 5,
         "tier": True, "bits": 1 << 16},
        # one aggregate kernel of the paper's width on a large dense state
        {"name": "block k5 29q c64", "kind": "block", "n": 29, "k": 5, "dtype": "c64"},
        # a two-qubit gate as it stands, no aggregation, odd size
        {"name": "block k2 25q c64", "kind": "block", "n": 25, "k": 2, "dtype": "c64"},
        # an aggregate gate in double
        {"name": "block k4 27q c128", "kind": "block", "n": 27, "k": 4, "dtype": "c128"},
        # a diagonal (hyperedge) gate on six qubits
        {"name": "diag m6 28q c64", "kind": "diag", "n": 28, "m": 6, "dtype": "c64"},
        # a change of layout on a resident state
        {"name": "permute 29q c64", "kind": "permute", "n": 29, "dtype": "c64"},
        # two tensors with four deferred bridging gates (eight entanglement indices)
        {"name": "contract 13+15 e8 c64", "kind": "contract", "n1": 13, "n2": 15, "e": 8, "dtype": "c64"},
        # the same in double, smaller parts
        {"name": "contract 12+13 e6 c128", "kind": "contract", "n1": 12, "n2": 13, "e": 6, "dtype": "c128"},
    ]


def draw(rng):
    kind = rng.choice(("circuit", "circuit", "batch", "sliced", "block", "block", "block", "diag", "permute",
                       "contract", "contract"))
    dtype = rng.choice(("c64", "c128"))
    if kind == "circuit":
        n = rng.randint(14, 28 if dtype == "c64" else 25)
        return {"kind": kind, "n": n, "depth": rng.randint(8, 20), "dtype": dtype, "kmax": rng.choice((4, 5)),
                "bits": 1 << rng.randint(8, min(n, 16)), "plan": "fast"}
    if kind == "batch":
        lo = rng.randint(16, 22)
        return {"kind": kind, "count": rng.randint(4, 24), "nmin": lo, "nmax": rng.randint(lo, 23), "dmin": 8,
                "dmax": rng.randint(8, 20), "bits": rng.choice((256, 1000, 1024))}
    if kind == "sliced":
        return {"kind": kind, "n": rng.choice(SLICED_N), "depth": rng.randint(8, 20), "dtype": dtype,
                "kmax": 5 if dtype == "c64" else 4, "tier": rng.random() < 0.5, "bits": 1 << rng.randint(8, 16)}
    if kind == "block":
        return {"kind": kind, "n": rng.randint(12, 29), "k": rng.randint(1, 6 if dtype == "c64" else 5),
                "dtype": dtype}
    if kind == "diag":
        return {"kind": kind, "n": rng.randint(12, 29), "m": rng.randint(1, 12), "dtype": dtype}
    if kind == "permute":
        return {"kind": kind, "n": rng.randint(12, 29), "dtype": dtype}
    return {"kind": kind, "n1": rng.randint(4, 13), "n2": rng.randint(4, 14), "e": rng.randint(1, 10), "dtype": dtype}


# ---- inputs --------------------------------------------------------------------

def circuit_of(case, seed):
    return W.sycamore_circuit(case["n"], case["depth"], seed=seed), W.bitstrings(case["n"], case["bits"], seed=seed + 1)


def batch_of(case, seed):
    """The batch's circuits and bitstrings: uneven sizes, the same sizes for every seed."""
    spec = np.random.default_rng(1004)
    ns = spec.integers(case["nmin"], case["nmax"] + 1, size=case["count"])
    ds = spec.integers(case["dmin"], case["dmax"] + 1, size=case["count"])
    return [(W.sycamore_circuit(int(n), int(d), seed=100 * seed + j),
             W.bitstrings(int(n), case["bits"], seed=100 * seed + 50 + j))
            for j, (n, d) in enumerate(zip(ns, ds))]


def gaussian(count, dtype, seed):
    """Complex normal values on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    real = torch.float32 if dtype == "c64" else torch.float64
    return torch.view_as_complex(torch.randn(count, 2, dtype=real, device="cuda", generator=g))


def dense_state(case, seed):
    """A normalised state with Porter-Thomas amplitudes, as deep random circuits have."""
    psi = gaussian(1 << case["n"], case["dtype"], seed)
    psi /= math.sqrt(2.0) * 2.0 ** (case["n"] / 2)
    return psi


def gate_of(case, seed):
    """Targets and entries of a random unitary block or a random diagonal gate."""
    rng = np.random.default_rng(seed)
    m = case["k"] if case["kind"] == "block" else case["m"]
    qubits = [int(q) for q in rng.choice(case["n"], size=m, replace=False)]
    entries = W.random_unitary(1 << m, rng) if case["kind"] == "block" else W.random_phases(1 << m, rng)
    return qubits, entries.astype(NUMPY[case["dtype"]])


def tensors_of(case, seed):
    t1 = gaussian(1 << (case["n1"] + case["e"]), case["dtype"], 2 * seed)
    t2 = gaussian(1 << (case["n2"] + case["e"]), case["dtype"], 2 * seed + 1)
    return t1, t2


class Program:
    """What a program keeps between calls: handles, plans and buffers."""

    def __init__(self, case):
        self.kind, self.dtype = case["kind"], case["dtype"] if "dtype" in case else "c64"
        self.handles, self.batch = [], None

    def __del__(self):
        try:
            if self.batch is not None:
                sv.batch_destroy(self.batch)
            for h in self.handles:
                sv.destroy_state(h)
        except Exception:                      # the interpreter is going down
            pass


class DeviceArray:
    """A device pointer of the library's as torch takes it; the tensor keeps its owner."""

    def __init__(self, owner, ptr, count, dtype):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<c%d" % AMP[dtype], "data": (ptr, False),
                                         "version": 2, "strides": None}


def view_of(program):
    """The amplitudes of a state the library allocated."""
    ptr, _ = sv.device_buffer(program.handles[0])
    return torch.as_tensor(DeviceArray(program, ptr, 1 << program.n, program.dtype), device="cuda")


def plan_of(case, circuit):
    n, dtype = case["n"], case["dtype"]
    stage = planner.stage_tmax(n, dtype)
    if case["plan"] == "fast" and stage:
        return stage, planner.plan_fast(circuit.gates, case["kmax"], nloc=n, sparse_start=True, tmax=stage)
    return stage, planner.plan(circuit.gates, case["kmax"], staged=stage > 0, nloc=max(n, stage + 9) if stage else None,
                               sparse_start=stage > 0, tmax=stage or None)


def prepare(case, seed):
    p = Program(case)
    kind = case["kind"]
    if kind == "circuit":
        circuit, p.bits = circuit_of(case, seed)
        stage, ops = plan_of(case, circuit)
        p.psi = torch.empty(1 << case["n"], dtype=TORCH[p.dtype], device="cuda")
        h = sv.create_state_ext(case["n"], 0, p.dtype, None, p.psi.data_ptr(), p.psi.numel() * AMP[p.dtype])
        p.handles.append(h)
        sv.set_option(h, sv.SV_OPT_STAGE, stage)
        p.ops = planner.pack(ops, p.dtype)
    elif kind == "batch":
        p.jobs = batch_of(case, seed)
        plans = []
        for circuit, _ in p.jobs:
            n, stage = circuit.n, planner.stage_tmax(circuit.n)
            p.handles.append(sv.create_state(n, 0, "c64"))
            sv.set_option(p.handles[-1], sv.SV_OPT_STAGE, stage)
            plans.append(planner.plan_fast(circuit.gates, 5, nloc=n, sparse_start=True, tmax=stage) if stage
                         else planner.plan(circuit.gates, 5, staged=False))
        for h, ops in zip(p.handles, plans):
            planner.enqueue(h, ops, "c64")
        p.batch = sv.batch_prepare(p.handles, graph=True)
        p.pool = ThreadPoolExecutor(max_workers=runner.REDUCE_THREADS)
        list(p.pool.map(lambda _: None, range(runner.REDUCE_THREADS)))
    elif kind == "sliced":
        circuit, p.bits = circuit_of(case, seed)
        sets = runner.grid_slice_sets(case["n"])
        sched = planner.phase_schedule(circuit, *sets, case["kmax"])
        first = sched.phases[0].sliced
        h = sv.create_state(case["n"], sum(1 << q for q in first), p.dtype, None, case["tier"])
        p.handles.append(h)
        if p.dtype == "c64":
            sv.set_option(h, sv.SV_OPT_STAGE, planner.stage_tmax(case["n"] - len(first)))
        p.phases = [(ph.order, planner.pack(ph.ops, p.dtype)) for ph in sched.phases]
        p.trailing = sched.trailing
    elif kind in ("block", "diag"):
        p.psi = dense_state(case, seed)
        p.qubits, p.entries = gate_of(case, seed)
        torch.cuda.synchronize()
        p.handles.append(sv.create_state_ext(case["n"], 0, p.dtype, None, p.psi.data_ptr(),
                                             p.psi.numel() * AMP[p.dtype], keep=True))
    elif kind == "permute":
        p.n = case["n"]
        h = sv.create_state(p.n, 0, p.dtype)
        p.handles.append(h)
        view = view_of(p)
        sv.sync_state(h)
        view.copy_(dense_state(case, seed))
        p.step = np.random.default_rng(seed).permutation(p.n).tolist()
        p.order = list(range(p.n))
        torch.cuda.synchronize()
    else:
        p.t1, p.t2 = tensors_of(case, seed)
        p.sizes = (case["n1"], case["n2"], case["e"])
        p.out = torch.empty(1 << (case["n1"] + case["n2"]), dtype=TORCH[p.dtype], device="cuda")
    return p


# ---- one pass --------------------------------------------------------------------

def kept(result, dtype):
    """Amplitudes and (norm, sum N p, sum ln N p) as a caller keeps them, in the state's precision."""
    amps, stats = result
    return {"amps": amps.astype(NUMPY[dtype], copy=False), "stats": np.array(stats, dtype=REAL[dtype])}


def run(p):
    if p.kind == "circuit":
        h = p.handles[0]
        sv.reset(h)
        planner.enqueue(h, p.ops, p.dtype)
        return {**kept(sv.reduce_slices(h, p.bits), p.dtype), "psi": p.psi}
    if p.kind == "batch":
        for h in p.handles:
            sv.reset(h)
        sv.batch_launch(p.batch)
        return [kept(r, "c64") for r in p.pool.map(lambda hj: sv.reduce_slices(hj[0], hj[1][1]),
                                                   zip(p.handles, p.jobs))]
    if p.kind == "sliced":
        h = p.handles[0]
        sv.reset(h)
        for order, ops in p.phases:
            sv.permute_qubits(h, order)
            planner.enqueue(h, ops, p.dtype)
        return kept(sv.reduce_slices(h, p.bits, p.trailing), p.dtype)
    if p.kind == "block":
        sv.apply_fused(p.handles[0], p.qubits, p.entries, p.dtype)
        sv.sync_state(p.handles[0])
        return p.psi
    if p.kind == "diag":
        sv.apply_diag(p.handles[0], p.qubits, p.entries, p.dtype)
        sv.sync_state(p.handles[0])
        return p.psi
    if p.kind == "permute":
        p.order = [p.order[i] for i in p.step]
        sv.permute_qubits(p.handles[0], p.order)
        return view_of(p)
    sv.contract(p.t1.data_ptr(), p.t2.data_ptr(), p.out.data_ptr(), *p.sizes, p.dtype,
                torch.cuda.current_stream().cuda_stream)
    return p.out


# ---- what a pass cannot do without ----------------------------------------------------

def circuit_work(circuit, amp, bits):
    """The state written once; every gate's complex dot products on every amplitude."""
    per_amp = sum(8 * (1 << g.k) - 2 for g in circuit.gates)
    return {"bytes": amp * 2.0 ** circuit.n + 24.0 * bits, "flops": per_amp * 2.0 ** circuit.n}


def work(case):
    kind = case["kind"]
    if kind in ("circuit", "sliced"):
        return circuit_work(circuit_of(case, 1)[0], AMP[case["dtype"]], case["bits"])
    if kind == "batch":
        each = [circuit_work(c, 8, case["bits"]) for c, _ in batch_of(case, 1)]
        return {key: sum(w[key] for w in each) for key in ("bytes", "flops")}
    amp = AMP[case["dtype"]]
    if kind == "contract":
        m, n, k = 1 << case["n2"], 1 << case["n1"], 1 << case["e"]
        return {"bytes": amp * (m * k + k * n + m * n), "flops": 8.0 * m * n * k}
    size = 1 << case["n"]
    per_amp = {"block": 8 * (1 << case.get("k", 0)) - 2, "diag": 6, "permute": 0}[kind]
    return {"bytes": 2.0 * amp * size, "flops": per_amp * size}


# ---- the same in 64 bits, plain torch ----------------------------------------------------

def split_dims(n, qubits):
    """psi's shape with one axis per target (highest qubit first), and each target's axis."""
    shape, axis, top = [], {}, n
    for q in sorted(qubits, reverse=True):
        shape += [1 << (top - q - 1), 2]
        axis[q] = len(shape) - 1
        top = q
    return shape + [1 << top], axis


def apply_gate(psi, n, qubits, matrix):
    """matrix (2^k x 2^k, index bit j = qubits[j]) on those qubits of psi (complex128)."""
    shape, axis = split_dims(n, qubits)
    src = [axis[q] for q in reversed(qubits)]
    dst = list(range(len(qubits)))
    front = torch.movedim(psi.view(shape), src, dst)
    moved = front.shape
    y = torch.as_tensor(matrix, dtype=torch.complex128, device="cuda") @ front.reshape(1 << len(qubits), -1)
    return torch.movedim(y.view(moved), dst, src).reshape(-1)


def simulate_exact(circuit):
    """The circuit on |0...0>, each single-qubit gate multiplied into the next gate on its qubit."""
    psi = torch.zeros(1 << circuit.n, dtype=torch.complex128, device="cuda")
    psi[0] = 1.0
    waiting = {}
    for g in circuit.gates:
        if g.k == 1:
            q = g.qubits[0]
            waiting[q] = g.matrix @ waiting.get(q, np.eye(2))
            continue
        lo, hi = (waiting.pop(q, np.eye(2)) for q in g.qubits)
        psi = apply_gate(psi, circuit.n, list(g.qubits), g.matrix @ np.kron(hi, lo))
    for q, m in waiting.items():
        psi = apply_gate(psi, circuit.n, [q], m)
    return psi


def read_exact(psi, n, bits):
    amps = psi[torch.from_numpy(bits.astype(np.int64)).cuda()]
    p = 2.0 ** n * (amps.real.square() + amps.imag.square())
    norm = torch.view_as_real(psi).square().sum()
    return {"amps": amps.cpu().numpy(),
            "stats": np.array([norm.item(), p.sum().item(), p.log().sum().item()])}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("circuit", "sliced"):
        circuit, bits = circuit_of(case, seed)
        psi = simulate_exact(circuit)
        out = read_exact(psi, circuit.n, bits)
        return {**out, "psi": psi} if kind == "circuit" else out
    if kind == "batch":
        return [read_exact(simulate_exact(c), c.n, bits) for c, bits in batch_of(case, seed)]
    if kind == "block":
        qubits, entries = gate_of(case, seed)
        return apply_gate(dense_state(case, seed).to(torch.complex128), case["n"], qubits,
                          entries.astype(np.complex128))
    if kind == "diag":
        qubits, entries = gate_of(case, seed)
        index = torch.arange(1 << case["n"], device="cuda")
        c = torch.zeros_like(index)
        for j, q in enumerate(qubits):
            c |= ((index >> q) & 1) << j
        phases = torch.from_numpy(entries.astype(np.complex128)).cuda()
        return dense_state(case, seed).to(torch.complex128) * phases[c]
    if kind == "permute":
        # bit p of the new index is bit order[p] of the old one
        psi, n = dense_state(case, seed).to(torch.complex128), case["n"]
        order = np.random.default_rng(seed).permutation(n).tolist()
        new = torch.arange(1 << n, device="cuda")
        old = torch.zeros_like(new)
        for p, q in enumerate(order):
            old |= ((new >> p) & 1) << q
        return psi[old]
    t1, t2 = (t.to(torch.complex128) for t in tensors_of(case, seed))
    n1, n2, e = case["n1"], case["n2"], case["e"]
    return (t2.view(1 << e, 1 << n2).t().contiguous() @ t1.view(1 << e, 1 << n1)).view(-1)
