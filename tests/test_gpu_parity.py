"""GPU parity: the HIP path (through the C-ABI) against the CPU oracle, on
the same seeded inputs.  Tolerances: rel-L2 <= 1e-4 for complex64 state
arithmetic, <= 1e-12 for complex128 (relative L2 over the returned
amplitudes).  Every call goes through libsv.so; nothing falls back."""
import math
import os

import numpy as np
import pytest

from oracle import brute
from oracle import oracle as orc
from paper_1910_09534_amd import planner, runner, sv
from paper_1910_09534_amd import workload as W

pytestmark = pytest.mark.gpu

TOL = {"c64": 1e-4, "c128": 1e-12}


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def state_from_numpy(psi: np.ndarray, dtype: str, slice_mask: int = 0):
    """Resident state whose buffer (a torch tensor) holds psi in the initial
    layout (unsliced qubits ascending, then sliced ones)."""
    torch = _torch()
    n = int(psi.size).bit_length() - 1
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    order = [q for q in range(n) if not (slice_mask >> q) & 1] + \
            [q for q in range(n) if (slice_mask >> q) & 1]
    phys = brute.permute_state(psi, n, order) if slice_mask else psi
    t = torch.from_numpy(phys.astype(np.complex64 if dtype == "c64" else np.complex128)).to("cuda")
    torch.cuda.synchronize()
    h = sv.create_state_ext(n, slice_mask, dtype, None, t.data_ptr(), t.numel() * t.element_size(),
                            keep=True)
    return h, t


def read_all(h, n):
    return sv.gather_amplitudes(h, np.arange(1 << n, dtype=np.uint64))


# ---- single operations on random states ---------------------------------------

@pytest.mark.parametrize("mfma", [0, 4])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("qs", [(0,), (5,), (11,), (1, 0), (3, 9), (0, 6, 2), (7, 1, 10, 4),
                                (2, 8, 0, 11, 5), (9, 3, 6, 0, 11, 1), (13, 12, 4, 7),
                                (1, 2, 3, 0, 13), (8, 9, 10, 11, 12, 13)])
def test_dense_single_op(dtype, qs, mfma):
    """One dense block on a random 14-qubit state, VALU (mfma=0) and matrix-core
    (mfma=4, used for k >= 4 with complex64) kernels."""
    if dtype == "c128" and len(qs) > 5:
        pytest.skip("complex128 blocks stop at k=5")
    if mfma and dtype == "c128":
        pytest.skip("matrix-core kernel covers complex64")
    # complex64 with mfma=4: k >= 4 runs on the matrix cores (staged through
    # LDS when a target is below position 4); k < 4 blocks with a target
    # below position 4 are widened to k = 4 and take the staged path too
    n = 14
    rng = np.random.default_rng(len(qs) * 100 + qs[0])
    psi = W.random_state(n, rng)
    u = W.random_unitary(1 << len(qs), rng)
    h, t = state_from_numpy(psi, dtype)
    try:
        sv.set_option(h, sv.SV_OPT_MFMA, mfma)
        sv.apply_fused(h, qs, u, dtype)
        got = read_all(h, n)
    finally:
        sv.destroy_state(h)
    ref = orc.apply_dense(psi.copy(), qs, u)
    assert orc.rel_l2(got, ref) <= TOL[dtype] * 0.1


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("fold", [True, False])
def test_diag_standalone_and_folded(dtype, fold):
    n = 13
    rng = np.random.default_rng(7)
    psi = W.random_state(n, rng)
    u = W.random_unitary(8, rng)
    d1 = W.random_phases(8, rng)
    d2 = W.random_phases(4, rng)
    h, t = state_from_numpy(psi, dtype)
    try:
        sv.set_option(h, sv.SV_OPT_FOLD_DIAG, 1 if fold else 0)
        sv.apply_fused(h, (4, 0, 9), u, dtype)
        sv.apply_diag(h, (12, 0, 5), d1, dtype)      # folded into the sweep above
        sv.apply_diag(h, (3, 10), d2, dtype)         # standalone
        got = read_all(h, n)
    finally:
        sv.destroy_state(h)
    ref = orc.apply_dense(psi.copy(), (4, 0, 9), u)
    orc.apply_diag(ref, (12, 0, 5), d1)
    orc.apply_diag(ref, (3, 10), d2)
    assert orc.rel_l2(got, ref) <= TOL[dtype] * 0.1


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_permute_resident(dtype):
    n = 11
    rng = np.random.default_rng(5)
    psi = W.random_state(n, rng)
    h, t = state_from_numpy(psi, dtype)
    order = [int(x) for x in rng.permutation(n)]
    try:
        sv.permute_qubits(h, order)
        assert sv.get_order(h, n) == order
        sv.sync_state(h)
        raw = t.cpu().numpy().astype(np.complex128)
        # physical buffer = the layout map of the logical state
        assert np.abs(raw - brute.permute_state(psi, n, order)).max() <= 1e-6
        # logical reads are unaffected; gates after a permute address logical qubits
        u = W.random_unitary(4, rng)
        sv.apply_fused(h, (order[0], order[7]), u, dtype)
        got = read_all(h, n)
    finally:
        sv.destroy_state(h)
    ref = orc.apply_dense(psi.copy(), (order[0], order[7]), u)
    assert orc.rel_l2(got, ref) <= TOL[dtype] * 0.1


# ---- whole circuits ---------------------------------------------------------------

def test_cfg1_all_amplitudes_c128():
    """4x4 grid, depth 8, complex128: all 65536 amplitudes within 1e-12."""
    c = W.config_circuit(1)
    bits = W.config_bitstrings(1)
    res = runner.simulate(c, bits, dtype="c128", kmax=4)
    ref = orc.simulate(c)
    assert orc.rel_l2(res["amps"], ref[bits.astype(np.int64)]) <= TOL["c128"]
    assert abs(res["norm"] - 1) < 1e-12


@pytest.mark.parametrize("kmax", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("mfma", [0, 4])
def test_circuit_c64_vs_oracle(kmax, fold, mfma):
    n, d = 20, 14
    c = W.sycamore_circuit(n, d, seed=2002)
    bits = W.bitstrings(n, 4096, seed=3)
    res = runner.simulate(c, bits, dtype="c64", kmax=kmax, fold_diag=fold, mfma=mfma)
    ref = orc.gather(orc.simulate(c), bits)
    assert orc.rel_l2(res["amps"], ref) <= TOL["c64"]
    assert abs(res["norm"] - 1) < 1e-4


@pytest.mark.parametrize("stage", [0, 9, 11, 12, 13])
def test_circuit_c64_staged_widths(stage):
    """The whole planned circuit (planner ordered for the tile width, deferred
    reset, folded norm) at every staged tile width, and without staging."""
    n, d = 20, 14
    c = W.sycamore_circuit(n, d, seed=2003)
    bits = W.bitstrings(n, 4096, seed=4)
    res = runner.simulate(c, bits, dtype="c64", kmax=5, stage=stage)
    ref_psi = orc.simulate(c)
    assert orc.rel_l2(res["amps"], orc.gather(ref_psi, bits)) <= TOL["c64"]
    assert abs(res["norm"] - orc.norm(ref_psi)) < 1e-5
    if stage:
        assert res["counters"]["staged_blocks"] > 0
    else:
        assert res["counters"]["staged_blocks"] == 0


def test_circuit_c128_k5():
    n = 18
    c = W.sycamore_circuit(n, 10, seed=44)
    bits = W.bitstrings(n, 2048, seed=4)
    res = runner.simulate(c, bits, dtype="c128", kmax=5)
    ref = orc.gather(orc.simulate(c), bits)
    assert orc.rel_l2(res["amps"], ref) <= TOL["c128"]


def test_stats_match_oracle():
    n = 16
    c = W.sycamore_circuit(n, 12, seed=9)
    bits = W.bitstrings(n, 5000, seed=10)
    res = runner.simulate(c, bits, dtype="c128", kmax=4)
    psi = orc.simulate(c)
    amps, (nrm, s1, s2) = orc.reduce_slices_ref(psi, (), None, bits)
    assert abs(res["norm"] - nrm) < 1e-12
    assert abs(res["xeb_sum"] - s1) < 1e-9 * abs(s1)
    assert abs(res["xeb_log_sum"] - s2) < 1e-9 * abs(s2)


# ---- slicing ----------------------------------------------------------------------

def test_sliced_resident_reduce_with_trailing():
    """Slices resident in HBM: out[x] = sum_t T[x_S, t] psi_t(x_L) equals the
    unsliced state with T applied to the sliced qubits."""
    n = 12
    rng = np.random.default_rng(12)
    S = (2, 7, 11)
    mask = sum(1 << q for q in S)
    c = W.sycamore_circuit(n, 6, seed=13)
    psi = orc.simulate(c)
    h, t = state_from_numpy(psi, "c128", slice_mask=mask)
    T = W.random_unitary(8, rng)
    bits = rng.integers(0, 1 << n, size=3000).astype(np.uint64)
    try:
        amps, stats = sv.reduce_slices(h, bits, T)
        gath = sv.gather_amplitudes(h, bits)
    finally:
        sv.destroy_state(h)
    ref, (nrm, s1, s2) = orc.reduce_slices_ref(psi, S, T, bits)
    assert orc.rel_l2(amps, ref) <= 1e-12
    assert abs(stats[0] - nrm) < 1e-12
    assert orc.rel_l2(gath, psi[bits.astype(np.int64)]) <= 1e-12


def test_external_buffer_alignment():
    """An external state buffer must be 16-byte aligned (staged passes move
    pairs of adjacent amplitudes with 16-byte accesses)."""
    torch = _torch()
    t = torch.zeros((1 << 10) + 2, dtype=torch.complex64, device="cuda")
    with pytest.raises(sv.SVError) as e:
        sv.create_state_ext(10, 0, "c64", None, t.data_ptr() + 8, (1 << 10) * 8)
    assert e.value.code == sv.SV_EINVAL
    h = sv.create_state_ext(10, 0, "c64", None, t.data_ptr() + 16, (1 << 10) * 8)
    sv.destroy_state(h)


def test_dense_on_sliced_qubit_rejected():
    _torch()
    h = sv.create_state(8, 1 << 3, "c64")
    try:
        with pytest.raises(sv.SVError) as e:
            sv.apply_fused(h, (3, 1), np.eye(4), "c64")
        assert e.value.code == sv.SV_ESLICED
        sv.apply_diag(h, (3, 1), np.ones(4), "c64")   # diagonal on a sliced qubit is fine
        with pytest.raises(sv.SVError) as e:
            sv.apply_fused(h, (1, 1), np.eye(4), "c64")
        assert e.value.code == sv.SV_EINVAL
        with pytest.raises(sv.SVError) as e:
            sv.permute_qubits(h, [0, 1, 2, 3, 4, 5, 6, 6])
        assert e.value.code == sv.SV_EINVAL
        with pytest.raises(sv.SVError) as e:
            sv.gather_amplitudes(h, np.array([256], dtype=np.uint64))
        assert e.value.code == sv.SV_EINVAL
        for opt, bad in ((sv.SV_OPT_STAGE, 8), (sv.SV_OPT_STAGE, 15), (sv.SV_OPT_STAGE, -1),
                         (sv.SV_OPT_MFMA, -1), (99, 1)):
            with pytest.raises(sv.SVError) as e:
                sv.set_option(h, opt, bad)
            assert e.value.code == sv.SV_EINVAL
        for good in (0, 9, 14):
            sv.set_option(h, sv.SV_OPT_STAGE, good)
        a = sv.gather_amplitudes(h, np.array([0, 1], dtype=np.uint64))
        assert abs(a[0] - 1) == 0 and a[1] == 0
    finally:
        sv.destroy_state(h)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [12, 14, 18])
def test_staged_multiblock_pass(n, dtype):
    """Runs of 4/5-qubit blocks sharing an LDS tile go through one staged HBM
    pass (complex64: split-fp16 form; complex128: FP64 form); the result
    equals one pass per block and the oracle."""
    rng = np.random.default_rng(n)
    psi = W.random_state(n, rng)
    ops = []
    for _ in range(12):
        k = int(rng.choice([2, 4, 5]))
        pool = list(range(min(n, 9)))          # overlapping sets: consecutive blocks share a tile
        qs = [int(x) for x in rng.choice(pool, size=k, replace=False)]
        ops.append((qs, W.random_unitary(1 << k, rng)))
    outs = {}
    for stage in (12, 0):
        h, t = state_from_numpy(psi, dtype)
        try:
            sv.set_option(h, sv.SV_OPT_STAGE, stage)
            for qs, u in ops:
                sv.apply_fused(h, qs, u, dtype)
            outs[stage] = read_all(h, n)
            cnt = sv.counters(h)
        finally:
            sv.destroy_state(h)
        if stage:
            assert cnt["staged_blocks"] >= 2, "no staged pass was formed"
    ref = psi.copy()
    for qs, u in ops:
        orc.apply_dense(ref, qs, u)
    tol = 1e-5 if dtype == "c64" else 1e-12
    assert orc.rel_l2(outs[12], ref) <= tol
    assert orc.rel_l2(outs[0], ref) <= tol
    assert orc.rel_l2(outs[12], outs[0]) <= (1e-6 if dtype == "c64" else 1e-13)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,tmax", [(12, 12), (14, 9), (15, 10), (17, 11), (18, 12), (13, 13), (19, 13),
                                    (14, 14), (21, 14)])
def test_staged_pass_any_positions(n, tmax, dtype):
    """Staged passes over blocks whose targets lie anywhere (no position
    limit), with tiles widened to the largest width allowed: equal to one
    pass per block and to the oracle; the widened tile still holds every
    block's targets."""
    rng = np.random.default_rng(100 + n)
    psi = W.random_state(n, rng)
    ops = []
    hi = list(range(4, n))
    # at most tmax - 4 distinct positions outside 0..3, spread over the range
    pool = [int(x) for x in rng.choice(hi, size=min(len(hi), tmax - 4), replace=False)] + [0, 1, 2, 3]
    for _ in range(10):
        k = int(rng.choice([4, 5]))
        qs = [int(x) for x in rng.choice(pool, size=k, replace=False)]
        ops.append((qs, W.random_unitary(1 << k, rng)))
    outs = {}
    for stage in (tmax, 0):
        h, t = state_from_numpy(psi, dtype)
        try:
            sv.set_option(h, sv.SV_OPT_STAGE, stage)
            for qs, u in ops:
                sv.apply_fused(h, qs, u, dtype)
            outs[stage] = read_all(h, n)
            cnt = sv.counters(h)
        finally:
            sv.destroy_state(h)
        if stage:
            assert cnt["staged_blocks"] >= 2, "no staged pass was formed"
    ref = psi.copy()
    for qs, u in ops:
        orc.apply_dense(ref, qs, u)
    tol = 1e-5 if dtype == "c64" else 1e-12
    assert orc.rel_l2(outs[tmax], ref) <= tol
    assert orc.rel_l2(outs[0], ref) <= tol
    assert orc.rel_l2(outs[tmax], outs[0]) <= (1e-6 if dtype == "c64" else 1e-13)


@pytest.mark.parametrize("n,stage,blocks", [
    # three 5-qubit blocks on 14 positions: the tile and matrices fill the 160 KiB exactly
    (18, 14, [[4, 6, 7, 9, 10], [12, 13, 15, 16, 17], [0, 6, 12, 17, 2]]),
    # eight 4-qubit blocks on 14 positions (the most blocks a pass takes)
    (18, 14, [[4, 6, 7, 9], [10, 12, 13, 15], [16, 17, 0, 4], [6, 10, 16, 1], [7, 12, 17, 2],
              [9, 13, 3, 4], [15, 16, 6, 7], [0, 1, 12, 17]]),
    # [5, 4, 4] on 13 positions: two workgroups' 80 KiB exactly
    (17, 13, [[4, 5, 7, 8, 10], [11, 12, 14, 15], [4, 11, 1, 2]]),
])
def test_staged_pass_full_lds(n, stage, blocks):
    """Runs whose tile and matrices fill the LDS budget exactly run as one
    staged pass and equal one sweep per block and the oracle."""
    rng = np.random.default_rng(7000 + n + len(blocks))
    psi = W.random_state(n, rng)
    ops = [(qs, W.random_unitary(1 << len(qs), rng)) for qs in blocks]
    outs = {}
    for st in (stage, 0):
        h, t = state_from_numpy(psi, "c64")
        try:
            sv.set_option(h, sv.SV_OPT_STAGE, st)
            for qs, u in ops:
                sv.apply_fused(h, qs, u, "c64")
            outs[st] = read_all(h, n)
            cnt = sv.counters(h)
        finally:
            sv.destroy_state(h)
        if st:
            assert cnt["staged_blocks"] == len(blocks) and cnt["dense_sweeps"] == 1, cnt
    ref = psi.copy()
    for qs, u in ops:
        orc.apply_dense(ref, qs, u)
    assert orc.rel_l2(outs[stage], ref) <= 1e-5
    assert orc.rel_l2(outs[stage], outs[0]) <= 1e-6


def test_sweep_profile_splits_kinds():
    """With timing on, staged passes and single sweeps are reported apart,
    with their launch counts and the arithmetic of their blocks."""
    n = 16
    rng = np.random.default_rng(5)
    h, t = state_from_numpy(W.random_state(n, rng), "c64")
    try:
        sv.set_option(h, sv.SV_OPT_TIMING, 1)
        blocks = [([4, 5, 6, 7, 8], 5), ([6, 7, 8, 9], 4), ([3, 9, 10, 11, 4], 5)]
        for qs, k in blocks:                 # one staged pass (tile 0..11)
            sv.apply_fused(h, qs, W.random_unitary(1 << k, rng), "c64")
        sv.sync_state(h)
        sv.apply_fused(h, [5, 13, 15], W.random_unitary(8, rng), "c64")    # single VALU sweep
        sv.sync_state(h)
        p = sv.sweep_profile(h)
        assert p["staged"]["count"] == 1 and p["sweep"]["count"] == 1
        # split-fp16 form (unitary blocks, measured bound): 24 2^k per amplitude
        assert sv.stage_forms(h)["split"] == 1
        assert p["staged"]["issued"] == 24.0 * (32 + 16 + 32) * (1 << n)
        assert p["staged"]["flops"] == (8.0 * 32 - 2 + 8.0 * 16 - 2 + 8.0 * 32 - 2) * (1 << n)
        assert p["sweep"]["issued"] == 8.0 * 8 * (1 << n)
        assert p["sweep"]["flops"] == (8.0 * 8 - 2) * (1 << n)
        assert p["staged"]["ms"] > 0 and p["sweep"]["ms"] > 0
        assert p["staged"]["bytes"] == 16.0 * (1 << n) and p["sweep"]["bytes"] == 16.0 * (1 << n)
        q = sv.sweep_profile(h)              # reset by the previous call
        assert q["staged"]["count"] == 0 and q["sweep"]["count"] == 0
        # from |0...0> the pass visits the one tile that can be non-zero and
        # reads nothing
        sv.reset(h)
        for qs, k in blocks:
            sv.apply_fused(h, qs, W.random_unitary(1 << k, rng), "c64")
        sv.sync_state(h)
        r = sv.sweep_profile(h)["staged"]
        visited = r["flops"] / (8.0 * 32 - 2 + 8.0 * 16 - 2 + 8.0 * 32 - 2)
        assert r["count"] == 1 and visited in (2.0 ** 12, 2.0 ** 13)
        assert r["bytes"] == 8.0 * visited
    finally:
        sv.destroy_state(h)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("count", [0, 1, 255, 257, (1 << 17), (1 << 17) + 1, 600_000])
def test_reduce_counts(count, dtype):
    """The one-launch reduction: no bitstrings, one workgroup, several, the
    largest call through pinned memory and the first one past it, more
    bitstrings than workgroups times lanes; two calls in a row.  Amplitudes
    are read exactly; the FP64 sums of at most 600,000 terms agree with
    numpy's within 1e-12."""
    n = 16
    rng = np.random.default_rng(count + 3)
    psi = W.random_state(n, rng).astype(np.complex64 if dtype == "c64" else np.complex128)
    h, t = state_from_numpy(psi, dtype)
    try:
        for rep in range(2):
            bits = W.bitstrings(n, count, seed=count + rep) if count else np.zeros(0, dtype=np.uint64)
            amps, stats = sv.reduce_slices(h, bits)
            ref = psi[bits.astype(np.int64)].astype(np.complex128)
            assert np.array_equal(amps, ref)
            p = 2.0 ** n * np.abs(ref) ** 2
            want = (np.sum(np.abs(psi.astype(np.complex128)) ** 2), np.sum(p), np.sum(np.log(p)))
            assert np.allclose(stats, want, rtol=1e-12, atol=1e-9), (stats, want)
            assert np.array_equal(sv.gather_amplitudes(h, bits), ref)
    finally:
        sv.destroy_state(h)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_reduce_resident_slices_with_trailing(dtype):
    """A resident state with sliced qubits: the sum over all slices in one
    launch, with and without a trailing operator, after a permute that
    changes the sliced set."""
    n, S = 13, (2, 7, 11)
    rng = np.random.default_rng(5)
    st = sv.State(n, sum(1 << q for q in S), dtype)
    try:
        psi = orc.zero_state(n)
        for q in range(n):
            if q not in S:
                u = W.random_unitary(2, rng)
                st.fused([q], u)
                orc.apply_dense(psi, [q], u)
        order = st.order()
        order[0], order[n - 1] = order[n - 1], order[0]
        st.permute(order)
        for q in order[:n - 3]:
            u = W.random_unitary(2, rng)
            st.fused([q], u)
            orc.apply_dense(psi, [q], u)
        sliced = sorted(order[n - 3:])
        T = rng.standard_normal((8, 8)) + 1j * rng.standard_normal((8, 8))
        bits = np.arange(1 << n, dtype=np.uint64)
        for trailing in (None, T):
            got, stats = st.reduce(bits, trailing)
            ref = psi.copy()
            if trailing is not None:
                orc.apply_dense(ref, sliced, trailing)
            assert orc.rel_l2(got, ref) <= TOL[dtype] * 0.1
            assert abs(stats[0] - 1.0) <= (1e-5 if dtype == "c64" else 1e-12)
    finally:
        st.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,sliced", [(1, 0), (2, 0), (7, 0), (8, 0), (9, 0), (10, 0), (14, 0), (14, 3), (11, 3)])
def test_diag_positions(n, sliced, dtype):
    """A diagonal gate on its own: positions inside an access (0), inside a
    workgroup's chunk, above it and sliced, in any order, up to 12 of them;
    states below and above one chunk.  One complex product per amplitude:
    2 eps."""
    rng = np.random.default_rng(1000 * n + sliced)
    mask = ((1 << sliced) - 1) << (n - sliced)
    sets = [[0], [n - 1], list(range(min(n, 12))), list(range(max(0, n - 12), n)),
            [int(q) for q in rng.choice(n, size=max(1, min(n, 12) // 2), replace=False)]]
    for qs in sets:
        qs = [int(q) for q in rng.permutation(qs)]
        st = sv.State(n, mask, dtype)
        try:
            psi = orc.zero_state(n)
            for q in range(n - sliced):                  # every local amplitude non-zero
                u = W.random_unitary(2, rng)
                st.fused([q], u)
                orc.apply_dense(psi, [q], u)
            before = read_all(st.h, n)
            ph = W.random_phases(1 << len(qs), rng)
            st.diag(qs, ph)
            got = read_all(st.h, n)
            ref = before.copy()
            orc.apply_diag(ref, qs, ph.astype(np.complex64) if dtype == "c64" else ph)
            assert orc.rel_l2(got, ref) <= (2.0 ** -23 if dtype == "c64" else 2.0 ** -52), qs
            assert sv.counters(st.h)["diag_sweeps"] == 1
        finally:
            st.close()


@pytest.mark.parametrize("n", [8, 9, 10, 14])
@pytest.mark.parametrize("k", [4, 5])
def test_dense64_matrix_core_sweep(n, k):
    """complex128 blocks of 4 and 5 qubits as single sweeps: one unit of 16
    groups in all (or too few: the vector form), a few, many; low, high and
    mixed targets in any order, alone and with a folded diagonal.  A sum of
    2^k products of a unitary's entries: 8 eps."""
    rng = np.random.default_rng(100 * n + k)
    for targets in (list(range(k)), list(range(n - k, n)), [int(x) for x in rng.choice(n, size=k, replace=False)]):
        for diag in (None, (0, n - 1, n // 2)):
            qs = [int(q) for q in rng.permutation(targets)]
            psi = W.random_state(n, rng)
            h, t = state_from_numpy(psi, "c128")
            try:
                sv.set_option(h, sv.SV_OPT_STAGE, 0)
                u = W.random_unitary(1 << k, rng)
                sv.apply_fused(h, qs, u, "c128")
                ref = psi.copy()
                orc.apply_dense(ref, qs, u)
                if diag:
                    ph = W.random_phases(8, rng)
                    sv.apply_diag(h, diag, ph, "c128")
                    orc.apply_diag(ref, list(diag), ph)
                assert orc.rel_l2(read_all(h, n), ref) <= 8 * 2.0 ** -52, (qs, diag)
                assert sv.counters(h)["dense_sweeps"] == 1 and sv.counters(h)["diag_sweeps"] == 0
            finally:
                sv.destroy_state(h)


@pytest.mark.parametrize("first", ["staged", "single", "read"])
def test_deferred_reset(first):
    """sv_reset defers writing |0...0>: a first staged pass builds its input
    from |0...0> without reading HBM, any other first use writes it first.
    The state is dirtied before the reset so a skipped write would show."""
    n = 14
    rng = np.random.default_rng(11)
    h, t = state_from_numpy(W.random_state(n, rng), "c64")
    try:
        for _ in range(3):                       # several resets in a row
            sv.reset(h)
            ops = []
            if first == "staged":
                ops = [([4, 5, 6, 7, 8], W.random_unitary(32, rng)), ([6, 7, 8, 9], W.random_unitary(16, rng)),
                       ([9, 10, 11, 4], W.random_unitary(16, rng))]
            elif first == "single":
                ops = [([5, 11], W.random_unitary(4, rng)), ([4, 5, 6, 7, 8], W.random_unitary(32, rng))]
            for qs, u in ops:
                sv.apply_fused(h, qs, u, "c64")
            got = read_all(h, n)
            ref = orc.zero_state(n)
            for qs, u in ops:
                orc.apply_dense(ref, qs, u)
            assert orc.rel_l2(got, ref) <= 1e-5
            # dirty the buffer again for the next round
            sv.apply_fused(h, [0, 1, 2], W.random_unitary(8, rng), "c64")
            sv.sync_state(h)
        if first == "staged":
            assert sv.counters(h)["staged_blocks"] >= 9
    finally:
        sv.destroy_state(h)


@pytest.mark.parametrize("case", ["read", "sweep", "diag", "chain", "chain-t11", "norm"])
def test_sparse_start_after_reset(case):
    """After sv_reset only the positions some operation has touched can hold
    non-zero amplitudes; staged passes visit only the tiles inside that
    support and take the never-written part of their tile as zero.  The
    buffer is dirtied before every reset, then the queue reads the state
    before every position is reached, runs a plain sweep or a diagonal in
    between, or reaches all positions pass by pass."""
    n = 20
    rng = np.random.default_rng(["read", "sweep", "diag", "chain", "chain-t11", "norm"].index(case) + 40)
    h, t = state_from_numpy(W.random_state(n, rng), "c64")
    if case == "chain-t11":
        sv.set_option(h, sv.SV_OPT_STAGE, 11)
    U = lambda k: W.random_unitary(1 << k, rng)
    try:
        for rep in range(2):
            sv.reset(h)
            c0 = sv.counters(h)["amps_swept"]
            ops = [("d", [4, 5, 6, 7, 8], U(5)), ("d", [5, 6, 7, 8, 9], U(5))]
            if case == "sweep":
                ops += [("d", [14, 16, 18], U(3))]
            if case == "diag":
                ops += [("g", [15, 17], np.exp(1j * rng.uniform(0, 6.3, 4)))]
            if case in ("sweep", "diag", "chain", "chain-t11"):
                ops += [("d", [13, 14, 15, 16], U(4)), ("d", [15, 16, 17, 18], U(4)),
                        ("d", [19, 4, 5, 6], U(4)), ("d", [18, 19, 2, 10], U(4))]
            for kind, qs, m in ops:
                if kind == "d":
                    sv.apply_fused(h, qs, m, "c64")
                else:
                    sv.apply_diag(h, qs, m, "c64")
            ref = orc.zero_state(n)
            for kind, qs, m in ops:
                if kind == "d":
                    orc.apply_dense(ref, qs, m)
                else:
                    orc.apply_diag(ref, qs, m)
            if case == "norm":
                bits = W.bitstrings(n, 256, seed=rep)
                amps, stats = sv.reduce_slices(h, bits)
                assert abs(stats[0] - orc.norm(ref)) <= 2e-6
                assert orc.rel_l2(amps, orc.gather(ref, bits)) <= 1e-5
            else:
                got = read_all(h, n)
                assert orc.rel_l2(got, ref) <= 1e-5
            if case.startswith("chain"):
                # the first two passes visit a fraction of the state only
                assert sv.counters(h)["amps_swept"] - c0 < 3 * (1 << n)
            # dirty the whole buffer for the next reset
            sv.apply_fused(h, [0, 1, 2], U(3), "c64")
            sv.sync_state(h)
    finally:
        sv.destroy_state(h)


@pytest.mark.parametrize("reset", [False, True])
def test_sparse_support_follows_permutes(reset):
    """A fresh (or reset) state is non-zero only on the positions its ops
    have targeted; a permute moves those positions with their qubits, and
    later staged passes visit the moved support."""
    n = 20
    rng = np.random.default_rng(70 + reset)
    U = lambda k: W.random_unitary(1 << k, rng)
    st = sv.State(n, 0, "c64")
    try:
        if reset:
            st.fused([0, 1, 2, 3, 4], U(5).astype(np.complex64))
            st.sync()
            sv.reset(st.h)
        ref = orc.zero_state(n)
        steps = [("f", [4, 5, 6, 7, 8], U(5)), ("f", [6, 7, 8, 9], U(4)),
                 ("p", [int(x) for x in rng.permutation(n)], None),
                 ("f", [7, 8, 15, 16], U(4)), ("f", [16, 17, 18, 19], U(4)),
                 ("p", list(range(n))[::-1], None),
                 ("f", [1, 2, 12, 19], U(4)), ("f", [9, 10, 11, 12, 13], U(5))]
        for kind, qs, m in steps:
            if kind == "f":
                st.fused(qs, m.astype(np.complex64))
                orc.apply_dense(ref, qs, m)
            else:
                st.permute(qs)
        got = st.gather(np.arange(1 << n, dtype=np.uint64))
    finally:
        st.close()
    assert orc.rel_l2(got, ref) <= 1e-5


@pytest.mark.parametrize("when", ["fresh", "reset", "reset-twice"])
def test_permute_of_zero_state_is_a_relabel(when):
    """A permute of a resident |0...0> with nothing queued moves no data (no
    permute sweep is counted) but takes the new layout: later operations,
    gathers and a second permute see the qubits where the layout put them.
    "reset" leaves stale values in the buffer, which must not show."""
    n = 18
    rng = np.random.default_rng(90 + len(when))
    U = lambda k: W.random_unitary(1 << k, rng)
    st = sv.State(n, 0, "c64")
    try:
        if when != "fresh":
            st.fused([0, 1, 2, 3, 4], U(5).astype(np.complex64))
            st.sync()
            sv.reset(st.h)
        p0 = sv.counters(st.h)["perm_sweeps"]
        st.permute([int(x) for x in rng.permutation(n)])
        if when == "reset-twice":
            st.permute(list(range(n))[::-1])
        assert sv.counters(st.h)["perm_sweeps"] == p0
        ref = orc.zero_state(n)
        for qs, k in (([3, 9, 14, 17], 4), ([0, 1, 2, 3, 4], 5), ([9, 10, 11, 12], 4)):
            m = U(k)
            st.fused(qs, m.astype(np.complex64))
            orc.apply_dense(ref, qs, m)
        st.permute(list(range(n)))           # the state is no longer |0...0>: data moves
        assert sv.counters(st.h)["perm_sweeps"] == p0 + 1
        got = st.gather(np.arange(1 << n, dtype=np.uint64))
    finally:
        st.close()
    assert orc.rel_l2(got, ref) <= 1e-5


@pytest.mark.parametrize("n,depth", [(20, 12), (22, 10), (24, 10)])
def test_sparse_start_plan_visits_as_modelled(n, depth):
    """A circuit planned for a run from |0...0> after sv_reset: the state
    equals the oracle's, and the amplitudes the passes visit equal the
    planner's model of the device (tile positions, widening inside the
    support, support growth), pass by pass in total."""
    from paper_1910_09534_amd import planner
    c = W.sycamore_circuit(n, depth, seed=60 + n)
    tmax = planner.stage_tmax(n)
    ops = planner.plan(c.gates, 5, sparse_start=True, nloc=n)
    rng = np.random.default_rng(n)
    h, t = state_from_numpy(W.random_state(n, rng), "c64")
    sv.set_option(h, sv.SV_OPT_STAGE, tmax)
    try:
        for _ in range(2):
            sv.reset(h)
            c0 = sv.counters(h)["amps_swept"]
            planner.enqueue(h, ops, sv.SV_C64)
            sv.sync_state(h)
            swept = sv.counters(h)["amps_swept"] - c0
            predicted = sum(1 << lv for _, lv in planner.sparse_passes(ops, n, None, tmax))
            assert swept == predicted
            assert swept < len(planner.stage_runs(ops, None, tmax)) * (1 << n)
            assert orc.rel_l2(read_all(h, n), orc.simulate(c)) <= 2e-5
    finally:
        sv.destroy_state(h)


@pytest.mark.parametrize("last,n", [("staged", 15), ("single", 15), ("single-dense", 15), ("staged", 23)])
def test_norm_folded_into_last_staged_pass(last, n):
    """When the queue ends with a staged pass, that pass also sums |psi|^2
    (FP64, per workgroup) and the reduction uses those sums; the norm and
    the amplitudes equal the oracle's either way.  At 23 qubits every
    workgroup takes two tiles (the second parked while the first is
    stored)."""
    rng = np.random.default_rng({"staged": 21, "single": 22, "single-dense": 23}[last] + n)
    psi = W.random_state(n, rng)
    h, t = state_from_numpy(psi, "c64")
    ops = [([4, 5, 6, 7, 8], W.random_unitary(32, rng)), ([6, 7, 8, 9], W.random_unitary(16, rng)),
           ([1, 9, 10, 14], W.random_unitary(16, rng))]
    if last == "single":              # promoted to 4 qubits: a one-block staged pass
        ops.append(([2, 13], W.random_unitary(4, rng)))
    if last == "single-dense":        # 3 qubits above position 3: a plain sweep, norm read after
        ops.append(([5, 11, 13], W.random_unitary(8, rng)))
    try:
        for qs, u in ops:
            sv.apply_fused(h, qs, u, "c64")
        bits = W.bitstrings(n, 512, seed=5)
        amps, stats = sv.reduce_slices(h, bits)
        ref = psi.astype(np.complex128).copy()
        for qs, u in ops:
            orc.apply_dense(ref, qs, u)
        assert abs(stats[0] - orc.norm(ref)) <= 2e-6
        assert orc.rel_l2(amps, orc.gather(ref, bits)) <= 1e-5
        if last == "staged":
            assert sv.counters(h)["staged_blocks"] >= 2
    finally:
        sv.destroy_state(h)


def test_headline_configuration_full_size():
    """The 30-qubit depth-14 workload in the launch configuration the
    benchmark times (resident complex64 state in a torch buffer, sv_reset,
    the plan for a run from |0...0>, staged passes, FP64 reduction of 2^16
    bitstrings), checked by properties that hold at any size: the norm is 1,
    the Porter-Thomas moments of the sampled probabilities (mean N p = 1,
    mean (N p)^2 = 2), two steps are bitwise identical, and the circuit
    followed by its inverse returns |0...0>."""
    torch = _torch()
    from paper_1910_09534_amd import planner
    circ = W.config_circuit(2)
    bits = W.config_bitstrings(2)
    n = circ.n
    ops = planner.plan(circ.gates, 5, sparse_start=True)
    inv = [W.Gate(g.qubits, np.conj(g.matrix).T) for g in reversed(circ.gates)]
    inv_ops = planner.plan(inv, 5)
    buf = torch.empty(1 << n, dtype=torch.complex64, device="cuda")
    h = sv.create_state_ext(n, 0, "c64", None, buf.data_ptr(), buf.numel() * 8)
    sv.set_option(h, sv.SV_OPT_STAGE, planner.stage_tmax(n))
    try:
        outs = []
        for _ in range(2):
            sv.reset(h)
            planner.enqueue(h, ops, sv.SV_C64)
            amps, stats = sv.reduce_slices(h, bits)
            outs.append(amps)
        assert np.array_equal(outs[0], outs[1])
        assert abs(stats[0] - 1.0) <= 1e-5
        p = (np.abs(outs[0]) ** 2) * float(1 << n)
        assert abs(p.mean() - 1.0) <= 0.03
        assert abs((p ** 2).mean() - 2.0) <= 0.2
        planner.enqueue(h, inv_ops, sv.SV_C64)          # U^-1 U |0...0>
        back = sv.gather_amplitudes(h, np.array([0, 1, 12345, (1 << n) - 1], dtype=np.uint64))
        assert abs(abs(back[0]) - 1.0) <= 1e-4
        assert np.abs(back[1:]).max() <= 1e-4
    finally:
        sv.destroy_state(h)
        del buf


@pytest.mark.parametrize("n", [18, 21])
def test_c128_staged_circuit_from_reset(n):
    """A planned circuit on a complex128 state through FP64 staged passes
    from a reset (the first pass builds its tiles from |0...0>, later ones
    take stale memory on newly reached positions as zero, the last one sums
    the norm), run twice so the second run starts over the first one's
    amplitudes: both equal the oracle to 1e-12, norm included."""
    _torch()
    circ = W.sycamore_circuit(n, 10, seed=900 + n)
    tmax = planner.stage_tmax(n, "c128")
    ops = planner.plan(circ.gates, 5, sparse_start=True, tmax=tmax)
    bits = W.bitstrings(n, 512, seed=n)
    ref = orc.simulate(circ)
    st = sv.State(n, 0, "c128")
    try:
        sv.set_option(st.h, sv.SV_OPT_STAGE, tmax)
        packed = planner.pack(ops, sv.SV_C128)
        for _ in range(2):
            sv.reset(st.h)
            planner.enqueue(st.h, packed, sv.SV_C128)
            amps, stats = sv.reduce_slices(st.h, bits)
            assert orc.rel_l2(amps, orc.gather(ref, bits)) <= 1e-12
            assert abs(stats[0] - 1.0) <= 1e-12
        cnt = sv.counters(st.h)
    finally:
        st.close()
    assert cnt["staged_blocks"] >= 4, cnt


@pytest.mark.parametrize("start", ["dense", "reset"])
@pytest.mark.parametrize("t", [9, 10, 11, 12, 13])
def test_c128_staged_block_forms(t, start):
    """4- and 5-qubit blocks as the only, first, middle and last block of an
    FP64 staged pass, on low, high and mixed targets, on every tile width, on
    a dense state and from a reset (tiles with unreached positions), the
    pass's norm included.  A block sums 32 products in each of three real
    products whose terms cancel by a factor of 3 at most: 2^-53 sqrt(32) 3,
    2e-15, with a factor 2.5 to spare: 5e-15 a block."""
    n = t + 5
    rng = np.random.default_rng(1300 + t)
    for ks in [(4,), (5,), (4, 5), (5, 4), (5, 5), (4, 4, 4), (5, 4, 5), (4, 5, 4), (4, 4, 5, 4)]:
        pool = [0, 1, 2, 3] + [int(x) for x in rng.choice(np.arange(4, n), size=5, replace=False)]
        psi = W.random_state(n, rng)
        h, tensor = state_from_numpy(psi, "c128")
        try:
            sv.set_option(h, sv.SV_OPT_STAGE, t)
            if start == "reset":
                sv.reset(h)
                psi = orc.zero_state(n)
            ref = psi.astype(np.complex128).copy()
            for k in ks:
                qs = [int(x) for x in rng.choice(pool, size=k, replace=False)]
                u = W.random_unitary(1 << k, rng)
                sv.apply_fused(h, qs, u, "c128")
                orc.apply_dense(ref, qs, u)
            got, stats = sv.reduce_slices(h, np.arange(1 << n, dtype=np.uint64))
            assert sv.counters(h)["staged_blocks"] >= 1
            assert orc.rel_l2(got, ref) <= 5e-15 * len(ks), (t, ks)
            assert abs(stats[0] - orc.norm(ref)) <= 1e-14 * len(ks)
        finally:
            sv.destroy_state(h)


@pytest.mark.parametrize("qs,diag", [([2, 9, 17, 24], None), ([0, 1, 2, 3, 4], [5, 24]), ([24, 11, 3, 20, 7], None),
                                     ([6, 0, 23, 12], [12, 1, 18])])
def test_dense64_large_state(qs, diag):
    """Complex128 sweeps on the matrix cores on a state beyond the last-level
    cache (non-temporal accesses), alone and with a folded diagonal, against
    the product done by torch in complex128: 2^-53 sqrt(32) for the sums with a
    factor 4 for the complex products on both sides."""
    torch = _torch()
    n, k = 25, len(qs)
    rng = np.random.default_rng(k + qs[0])
    g = torch.Generator(device="cuda").manual_seed(n + k)
    psi = torch.view_as_complex(torch.randn((1 << n, 2), generator=g, device="cuda", dtype=torch.float64))
    psi /= torch.linalg.vector_norm(psi)
    u = W.random_unitary(1 << k, rng)
    axes = [n - 1 - q for q in reversed(qs)]                    # matrix bit j = qubit qs[j]
    x = torch.movedim(psi.view([2] * n), axes, list(range(k))).reshape(1 << k, -1)
    ref = torch.from_numpy(u).cuda() @ x
    ref = torch.movedim(ref.view([2] * n), list(range(k)), axes).reshape(-1)
    if diag:
        ph = W.random_phases(1 << len(diag), rng)
        idx = torch.arange(1 << n, device="cuda")
        c = sum(((idx >> q) & 1) << j for j, q in enumerate(diag))
        ref = ref * torch.from_numpy(ph).cuda()[c]
    torch.cuda.synchronize()
    h = sv.create_state_ext(n, 0, "c128", None, psi.data_ptr(), psi.numel() * 16, keep=True)
    try:
        sv.apply_fused(h, qs, u, "c128")
        if diag:
            sv.apply_diag(h, diag, ph, "c128")
        sv.sync_state(h)
    finally:
        sv.destroy_state(h)
    assert float(torch.linalg.vector_norm(psi - ref)) <= 8 * 2.0 ** -53 * np.sqrt(32)


@pytest.mark.parametrize("n,dtype", [(25, "c64"), (26, "c64"), (24, "c128"), (25, "c128")])
def test_diag_large_state(n, dtype):
    """Diagonal gates on both sides of the size up to which a state's lanes
    read the table themselves, with few, all and none of a workgroup's positions
    taken.  One complex product per amplitude: 2 eps."""
    import torch

    rng = np.random.default_rng(n)
    real = torch.float32 if dtype == "c64" else torch.float64
    gen = torch.Generator(device="cuda").manual_seed(n)
    psi = torch.randn(1 << n, 2, dtype=real, device="cuda", generator=gen)
    index = torch.arange(1 << n, device="cuda", dtype=torch.int32)
    torch.cuda.synchronize()
    chunk = 9 if dtype == "c64" else 8
    for qs in ([0, 3, n - 1], list(range(chunk)) + [12, n - 1], list(range(chunk, chunk + 4)),
               list(range(1, 12))):
        qs = [int(q) for q in rng.permutation(qs)]
        before = psi.clone()
        torch.cuda.synchronize()
        h = sv.create_state_ext(n, 0, dtype, None, psi.data_ptr(), psi.numel() * psi.element_size(), keep=True)
        try:
            ph = W.random_phases(1 << len(qs), rng)
            sv.apply_diag(h, qs, ph, dtype)
            sv.sync_state(h)
        finally:
            sv.destroy_state(h)
        at = torch.zeros_like(index)
        for j, q in enumerate(qs):
            at |= ((index >> q) & 1) << j
        table = torch.from_numpy(ph.astype(np.complex64) if dtype == "c64" else ph).cuda().to(torch.complex128)
        ref = torch.view_as_complex(before.double()) * table[at.long()]
        got = torch.view_as_complex(psi.double())
        rel = ((got - ref).abs().square().sum() / ref.abs().square().sum()).sqrt().item()
        assert rel <= (2.0 ** -23 if dtype == "c64" else 2.0 ** -52), qs


@pytest.mark.parametrize("k", [4, 5])
def test_dense64_error_against_long_double(k):
    """A complex128 matrix-core sweep's error against 80-bit sums is no larger
    than that of adding the products one after the other in double (four real
    sums of half the length each)."""
    n = 14
    rng = np.random.default_rng(70 + k)
    psi = W.random_state(n, rng)
    qs = [int(q) for q in rng.choice(n, k, replace=False)]
    u = W.random_unitary(1 << k, rng)
    axes = [n - 1 - q for q in reversed(qs)]                    # matrix bit j = qubit qs[j]

    def one_after_the_other(dtype):
        x = np.moveaxis(psi.astype(dtype).reshape([2] * n), axes, range(k)).reshape(1 << k, -1)
        y = np.zeros_like(x)
        for j in range(1 << k):
            y += u[:, j:j + 1].astype(dtype) * x[j]
        return np.moveaxis(y.reshape([2] * n), range(k), axes).reshape(-1)

    h, t = state_from_numpy(psi, "c128")
    try:
        sv.set_option(h, sv.SV_OPT_STAGE, 0)
        sv.apply_fused(h, qs, u, "c128")
        got = read_all(h, n)
    finally:
        sv.destroy_state(h)
    exact = one_after_the_other(np.clongdouble)
    error = lambda x: float(np.linalg.norm((x - exact).astype(np.complex128)))
    assert error(got) <= error(one_after_the_other(np.complex128))
