"""GPU checks of the batched execution: many circuits of different qubit
counts in one graph-captured launch sequence.  Each result equals the same
plan run alone (bitwise), and the oracle (rel-L2 <= 1e-4 complex64,
<= 1e-12 complex128)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1910_09534_amd import planner, runner, sv
from paper_1910_09534_amd import workload as W

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _batch(count=10, nmin=12, nmax=20, seed=5):
    specs = W.batch_specs(count, seed=seed, nmin=nmin, nmax=nmax, dmin=6, dmax=12)
    circs = [W.sycamore_circuit(s["n"], s["depth"], s["seed"]) for s in specs]
    bits = [W.bitstrings(s["n"], 1024, s["bit_seed"]) for s in specs]
    return circs, bits


@pytest.mark.parametrize("graph", [True, False])
def test_batch_equals_alone_and_oracle(graph):
    _gpu()
    circs, bits = _batch()
    kmax = {n: (4 if n % 2 else 5) for n in range(12, 21)}
    plans = [planner.plan(c.gates, kmax[c.n], staged=False) for c in circs]
    res = runner.run_batch(circs, bits, "c64", kmax=kmax, graph=graph, repeats=2, plans=plans)
    assert res["info"]["graph"] == graph
    for c, b, amps, p in zip(circs, bits, res["amps"], plans):
        st = sv.State(c.n, 0, "c64")
        try:
            sv.set_option(st.h, sv.SV_OPT_STAGE, 0)          # as in the batch: no staged passes
            planner.enqueue(st.h, p, st.dtype)
            alone = st.gather(b)
        finally:
            st.close()
        assert np.array_equal(alone, amps), "batched result differs from the same plan alone"
        ref = orc.gather(orc.simulate(c), b)
        assert orc.rel_l2(amps, ref) <= 1e-4


@pytest.mark.parametrize("graph", [True, False])
def test_staged_batch_equals_alone_and_oracle(graph):
    """States of 2^18..2^21 amplitudes with staged passes in the batch (tile
    limit n - 9): each equals the same plan and tile limit alone (bitwise)
    and the oracle; replays after sv_reset give the same result."""
    _gpu()
    circs, bits = _batch(count=6, nmin=18, nmax=21, seed=13)
    res = runner.run_batch(circs, bits, "c64", kmax=5, graph=graph, repeats=2, staged=True)
    plans = [planner.plan_fast(c.gates, 5, nloc=c.n, sparse_start=True) for c in circs]
    staged_blocks = 0
    for c, b, amps, p in zip(circs, bits, res["amps"], plans):
        st = sv.State(c.n, 0, "c64")
        try:
            sv.set_option(st.h, sv.SV_OPT_STAGE, planner.stage_tmax(c.n))
            planner.enqueue(st.h, p, st.dtype)
            alone = st.gather(b)
            staged_blocks += sv.counters(st.h)["staged_blocks"]
        finally:
            st.close()
        assert np.array_equal(alone, amps), "batched result differs from the same plan alone"
        ref = orc.gather(orc.simulate(c), b)
        assert orc.rel_l2(amps, ref) <= 1e-4
    assert staged_blocks > 0


@pytest.mark.parametrize("graph", [True, False])
def test_batch_reset_variant(graph):
    """States all reset before the launch run the batch's reset variant:
    staged passes from |0...0> that visit only the tiles inside each state's
    support, |0...0> written only ahead of a plain sweep, and the part of the
    state no pass reached cleared at the end.  Covers a plain sweep early in
    a plan, a state with no ops, a state whose support stays partial, and a
    planned circuit; the buffers hold the previous run's values at every
    reset.  A launch without a reset runs the ordinary variant on the
    current states (the ops applied twice)."""
    _gpu()
    rng = np.random.default_rng(17)
    U = lambda k: W.random_unitary(1 << k, rng)
    c = W.sycamore_circuit(20, 10, seed=71)
    specs = [
        (18, 9, [([4, 5, 6, 7, 8], U(5)), ([5, 6, 7, 8, 9], U(5)), ([15, 16, 17], U(3)),
                 ([10, 11, 12, 13], U(4)), ([12, 13, 14, 15], U(4))]),
        (19, 10, []),
        (18, 9, [([14, 15, 16], U(3)), ([4, 5, 6, 7], U(4)), ([6, 7, 8, 9], U(4))]),
        (22, 13, [([0, 1, 2, 3, 4], U(5)), ([2, 3, 4, 5, 6], U(5)), ([6, 7, 8, 9], U(4))]),
        (20, 11, [(list(o.qubits), o.matrix) for o in
                  planner.plan_fast(c.gates, 5, nloc=20, sparse_start=True)]),
    ]
    states, b = [], None
    try:
        for n, tmax, ops in specs:
            st = sv.State(n, 0, "c64")
            sv.set_option(st.h, sv.SV_OPT_STAGE, tmax)
            for qs, m in ops:
                st.fused(qs, np.asarray(m).astype(np.complex64))
            states.append(st)
        b = sv.batch_prepare([st.h for st in states], graph=graph)
        refs = []
        for n, _, ops in specs:
            psi = orc.zero_state(n)
            for qs, m in ops:
                orc.apply_dense(psi, qs, m)
            refs.append(psi)
        for rep in range(3):
            for st in states:
                sv.reset(st.h)
            sv.batch_launch(b)
            for st, (n, _, _), ref in zip(states, specs, refs):
                got = st.gather(np.arange(1 << n, dtype=np.uint64))
                assert orc.rel_l2(got, ref) <= 1e-4, (n, rep)
        info_reset = sv.batch_info(b)
        # no reset: the batch applies its ops to the states as they are
        sv.batch_launch(b)
        info_plain = sv.batch_info(b)
        assert info_reset["amps_swept"] < info_plain["amps_swept"]
        assert info_reset["sweeps"] == info_plain["sweeps"]
        for st, (n, _, ops), ref in zip(states, specs, refs):
            twice = ref.copy()
            for qs, m in ops:
                orc.apply_dense(twice, qs, m)
            got = st.gather(np.arange(1 << n, dtype=np.uint64))
            assert orc.rel_l2(got, twice) <= 2e-4, n
    finally:
        if b is not None:
            sv.batch_destroy(b)
        for st in states:
            st.close()


def test_batch_c128_vs_c64_vs_oracle():
    _gpu()
    circs, bits = _batch(count=6, nmin=10, nmax=16, seed=9)
    r64 = runner.run_batch(circs, bits, "c64", kmax=5)
    r128 = runner.run_batch(circs, bits, "c128", kmax=4)
    for c, b, a64, a128, s128 in zip(circs, bits, r64["amps"], r128["amps"], r128["stats"]):
        ref = orc.gather(orc.simulate(c), b)
        assert orc.rel_l2(a128, ref) <= 1e-12
        assert orc.rel_l2(a64, a128) <= 1e-4
        assert abs(s128[0] - 1) < 1e-12


def test_batch_rejects_bad_inputs():
    _gpu()
    a = sv.State(10, 0, "c64")
    c = sv.State(10, 0, "c128")
    t = sv.State(10, 1 << 9, "c64", tier=True)
    try:
        with pytest.raises(sv.SVError):
            sv.batch_prepare([a.h, c.h])          # mixed dtypes
        with pytest.raises(sv.SVError):
            sv.batch_prepare([a.h, a.h])          # duplicate
        with pytest.raises(sv.SVError):
            sv.batch_prepare([a.h, t.h])          # tiered state
        # a state re-laid out after the batch was prepared is refused at launch
        u = W.random_unitary(4, np.random.default_rng(2)).astype(np.complex64)
        a.fused([0, 1], u)
        b = sv.batch_prepare([a.h])
        try:
            a.fused([2, 3], u)
            a.sync()
            a.permute(list(range(10))[::-1])
            with pytest.raises(sv.SVError):
                sv.batch_launch(b)
        finally:
            sv.batch_destroy(b)
    finally:
        a.close(); c.close(); t.close()


def test_tuned_staged_batch_matches_c128_batch_and_oracle():
    """The staged batch with the fusion width and tile limit chosen per qubit
    count by the autotuner (timed on this GPU): every result within the
    complex64 tolerance of the complex128 batch of the same circuits and of
    the oracle; the tuned choices are among the candidates."""
    _gpu()
    from paper_1910_09534_amd import autotune
    tuned = autotune.tune_staged([19, 21], kmaxes=(4, 5, 6), tiles=(10, 12), depth=8, reps=1)
    assert set(tuned["kmax"].values()) <= {4, 5, 6} and set(tuned["stage_t"].values()) <= {10, 12}
    pairs = [(c, b) for c, b in zip(*_batch(count=8, nmin=19, nmax=21, seed=29)) if c.n in (19, 21)]
    assert pairs
    circs, bits = [p[0] for p in pairs], [p[1] for p in pairs]
    res = runner.run_batch(circs, bits, "c64", kmax=tuned["kmax"], graph=True, repeats=2, staged=True,
                           stage_t=tuned["stage_t"])
    r128 = runner.run_batch(circs, bits, "c128", kmax=4, graph=True)
    for c, b, a64, a128 in zip(circs, bits, res["amps"], r128["amps"]):
        assert orc.rel_l2(a64, a128) <= 1e-4
        ref = orc.gather(orc.simulate(c), b)
        assert orc.rel_l2(a128, ref) <= 1e-12
        assert orc.rel_l2(a64, ref) <= 1e-4


@pytest.mark.parametrize("graph", [True, False])
def test_batch_c128_blocks_with_and_without_diagonals(graph):
    """Complex128 blocks of 4 and 5 qubits, plain and with a diagonal folded in,
    as batched matrix-core sweeps (one unit, several, and many a wave) and as
    vector sweeps below their size: each state has the bits of the same
    operations alone, and the oracle's amplitudes.  A block's 2^k-term dot
    products and a phase: sqrt(2^k) + 2 eps, k = 5 and 4 operations, factor 4."""
    _gpu()
    rng = np.random.default_rng(61)
    states, alone, refs, b = [], [], [], None
    try:
        for n in (7, 8, 9, 10, 13, 17, 19):
            ops = []
            for k, m in ((4, 0), (5, 3), (4, 2), (5, 0)):
                ops.append(("fused", [int(q) for q in rng.choice(n, k, replace=False)], W.random_unitary(1 << k, rng)))
                if m:
                    ops.append(("diag", [int(q) for q in rng.choice(n, m, replace=False)], W.random_phases(1 << m, rng)))
            pair = [sv.State(n, 0, "c128") for _ in range(2)]
            for st in pair:
                sv.set_option(st.h, sv.SV_OPT_STAGE, 0)              # as in the batch: no staged passes
                for kind, qs, m in ops:
                    (sv.apply_fused if kind == "fused" else sv.apply_diag)(st.h, qs, m, "c128")
            states.append(pair[0])
            alone.append(pair[1])
            psi = orc.zero_state(n)
            for kind, qs, m in ops:
                orc.apply_dense(psi, qs, m if kind == "fused" else np.diag(m))
            refs.append(psi)
        b = sv.batch_prepare([st.h for st in states], graph=graph)
        sv.batch_launch(b)
        for st, a, ref in zip(states, alone, refs):
            bits = np.arange(ref.size, dtype=np.uint64)
            got = st.gather(bits)
            assert np.array_equal(got, a.gather(bits)), ref.size
            assert orc.rel_l2(got, ref) <= 4 * 4 * (np.sqrt(32) + 2) * 2.0 ** -53, ref.size
    finally:
        if b is not None:
            sv.batch_destroy(b)
        for st in states + alone:
            st.close()


def test_batch_of_wide_and_small_states_side_by_side():
    """A state of 23 qubits (six graphs side by side) beside small ones that
    share launches with one another and with it: from a reset, applied again
    to what is there, and with only some of the states reset."""
    _gpu()
    rng = np.random.default_rng(67)
    U = lambda k: W.random_unitary(1 << k, rng)
    sizes = (23, 14, 12, 13, 20, 12, 15, 21)
    plans = []
    for i, n in enumerate(sizes):
        pick = lambda k: [int(q) for q in rng.choice(np.arange(4, n), k, replace=False)]
        ops = [(pick(5), U(5)), (pick(4), U(4))]
        if i not in (4, 7):                                  # shared vector sweeps of one and two widths
            ops.insert(1 if i % 2 else 2, (pick(3), U(3)))
        if i % 3 == 0:
            ops.append((pick(2), U(2)))
        plans.append(ops)
    states, b = [], None

    def applied(psi, ops):
        for qs, m in ops:
            orc.apply_dense(psi, qs, m)
        return psi

    def check(refs, tol):
        for st, ref, n in zip(states, refs, sizes):
            bits = W.bitstrings(n, 4096, seed=n)
            assert orc.rel_l2(st.gather(bits), orc.gather(ref, bits)) <= tol, n
    try:
        for n, ops in zip(sizes, plans):
            st = sv.State(n, 0, "c64")
            sv.set_option(st.h, sv.SV_OPT_STAGE, 12 if n >= 20 else 9)
            for qs, m in ops:
                st.fused(qs, np.asarray(m).astype(np.complex64))
            states.append(st)
        b = sv.batch_prepare([st.h for st in states], graph=True)
        for st in states:
            sv.reset(st.h)
        sv.batch_launch(b)
        refs = [applied(orc.zero_state(n), ops) for n, ops in zip(sizes, plans)]
        check(refs, 1e-5)
        sv.batch_launch(b)
        refs = [applied(ref, ops) for ref, ops in zip(refs, plans)]
        check(refs, 2e-5)
        for i in (0, 2, 5):
            sv.reset(states[i].h)
            refs[i] = orc.zero_state(sizes[i])
        sv.batch_launch(b)
        refs = [applied(ref, ops) for ref, ops in zip(refs, plans)]
        check(refs, 3e-5)
    finally:
        if b is not None:
            sv.batch_destroy(b)
        for st in states:
            st.close()
