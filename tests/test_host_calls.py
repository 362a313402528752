"""The library's host side on a machine without a GPU: libsv.so in a process
of its own whose HIP calls go to the stand-in runtime of fake_hip.cpp.  What
the stand-in sees is checked: launches within HIP's documented limits at every
size that fits the device, and what is still running when a call fails.  No
kernel runs, so results are the GPU tests' matter."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PRELUDE = """
import ctypes, sys
F = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)     # ahead of libsv.so's own runtime
F.fake_log.restype = ctypes.c_char_p
import numpy as np
from paper_1910_09534_amd import sv

def log():
    return F.fake_log().decode().splitlines()

def unitary(k, seed=0):
    r = np.random.default_rng(seed)
    return np.linalg.qr(r.normal(size=(2 ** k, 2 ** k)) + 1j * r.normal(size=(2 ** k, 2 ** k)))[0]

def code_of(f, *a):
    try:
        f(*a)
    except sv.SVError as e:
        return e.code
    return sv.SV_OK
"""


@pytest.fixture(scope="session")
def fake_hip(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(ROCM, "include"), os.path.join(HERE, "fake_hip.cpp"), "-o", out])
    return out


def run(fake_hip, body):
    p = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), fake_hip], cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout[-4000:] + p.stderr[-4000:]


@pytest.mark.parametrize("dtype,sizes", [("c64", (1, 5, 12, 30, 32, 33, 34)), ("c128", (1, 5, 12, 30, 31, 32, 33))])
def test_resident_operations_at_every_size(fake_hip, dtype, sizes):
    """Every operation of a resident state is launched, up to the states that
    fill the device (a launch takes fewer than 2^32 work items)."""
    run(fake_hip, f"""
    for n in {sizes}:
        for op in ("diag1", "diag3", "k1", "k2", "k3", "k4", "k5", "permute", "reduce"):
            h = sv.create_state(n, 0, "{dtype}")
            if op.startswith("diag"):
                q = sorted({{0, n // 2, n - 1}})[:int(op[4])]
                sv.apply_diag(h, q, np.ones(1 << len(q)), "{dtype}")
            elif op.startswith("k"):
                k = min(int(op[1]), n)
                sv.apply_fused(h, list(range(n - k, n)), unitary(k), "{dtype}")
            elif op == "permute":
                sv.apply_fused(h, [0], unitary(1), "{dtype}")
                if n <= 30:
                    sv.sync_state(h)
                    sv.permute_qubits(h, list(range(n))[::-1])
            else:
                sv.reduce_slices(h, np.arange(2, dtype=np.uint64))
            sv.sync_state(h)
            sv.destroy_state(h)
    assert not [x for x in log() if x.startswith("refused")]
    """)


@pytest.mark.parametrize("dtype,n", [("c64", 32), ("c64", 33), ("c64", 34), ("c128", 33)])
def test_diagonal_covers_large_states(fake_hip, dtype, n):
    """The workgroups of a diagonal gate's launches cover the state once."""
    run(fake_hip, f"""
    h = sv.create_state({n}, 0, "{dtype}")
    F.fake_clear()
    sv.apply_diag(h, [0, 9, {n} - 1], np.ones(8), "{dtype}")
    sv.sync_state(h)
    grids = [int(x.split(" grid ")[1].split()[0]) for x in log() if x.startswith("launch") and "k_diag" in x]
    assert sum(grids) * 256 * (2 if "{dtype}" == "c64" else 1) == 1 << {n}, grids
    """)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_contractions_at_every_size(fake_hip, dtype):
    """Every contraction that fits the device is launched, in both forms."""
    run(fake_hip, f"""
    amp = 8 if "{dtype}" == "c64" else 16
    at = 1 << 44                                    # (never read: no kernel runs)
    for n1 in range(36):
        for n2 in range(36):
            for e in range(13):
                if amp * (2 ** (n1 + n2) + 2 ** (n1 + e) + 2 ** (n2 + e)) > 288e9:
                    continue
                for fp32 in (False, True) if amp == 8 else (False,):
                    code = code_of(lambda: sv.contract(at, 2 * at, 3 * at, n1, n2, e, "{dtype}", fp32=fp32))
                    assert code == sv.SV_OK, (n1, n2, e, fp32)
    """)


@pytest.mark.parametrize("api", ["hipMemcpyAsync", "hipEventRecord"])
def test_failed_call_leaves_other_handles(fake_hip, api):
    """A runtime call that fails is told by the call that made it: its handle
    is unusable from then on, another one's next launch does not fail for it."""
    run(fake_hip, f"""
    a, b, c = (sv.create_state(12, 0, "c64") for _ in range(3))
    batch = sv.batch_prepare([a], graph=False)
    if "{api}" == "hipMemcpyAsync":
        F.fake_fail(b"{api}", 1)
        assert code_of(sv.reduce_slices_noalloc, a, np.arange(4, dtype=np.uint64)) == sv.SV_EDEVICE
        assert code_of(sv.sync_state, a) == sv.SV_ESTATE
    else:
        F.fake_fail(b"{api}", 1)
        assert code_of(sv.batch_launch, batch) == sv.SV_EDEVICE
    sv.apply_diag(b, [0], np.ones(2), "c64")
    assert code_of(sv.sync_state, b) == sv.SV_OK
    sv.reduce_slices(c, np.arange(4, dtype=np.uint64))
    """)


BATCH = """
def batch(graph, sizes=(20, 21, 22, 20, 23, 12)):
    hs = [sv.create_state(n, 0, "c64") for n in sizes]
    for h in hs:
        for q in range(0, 10, 5):
            sv.apply_fused(h, list(range(q, q + 5)), unitary(5), "c64")
    b = sv.batch_prepare(hs, graph=graph)
    for h in hs:
        sv.sync_state(h)
    assert F.fake_undone() == 0
    return hs, b
"""


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("api", ["hipGraphLaunch", "hipLaunchKernel", "hipEventRecord", "hipStreamWaitEvent"])
def test_batch_launch_that_fails(fake_hip, api, graph):
    """However far a batch launch gets before a runtime call fails, nothing of
    it runs on when it returns (the caller may free the states), and no state
    is half of one thing: usable as it was before, or refused."""
    run(fake_hip, BATCH + textwrap.dedent(f"""
    bits = np.arange(4, dtype=np.uint64)
    failed = 0
    for nth in range(1, 40):
        hs, b = batch({graph})
        for h in hs:
            sv.reset(h)
        F.fake_fail(b"{api}", nth)
        F.fake_clear()
        code = code_of(sv.batch_launch, b)
        ran = any(x.startswith(("graph", "launch")) for x in log())
        F.fake_fail(b"{api}", 0)                                  # (not reached: off)
        if code == sv.SV_OK:
            for h in hs:
                sv.destroy_state(h)
            sv.batch_destroy(b)
            continue
        failed += 1
        assert F.fake_undone() == 0, nth
        for h in hs:
            if ran:
                assert code_of(sv.reduce_slices, h, bits) == sv.SV_ESTATE, nth
            else:
                F.fake_clear()
                if code_of(sv.reduce_slices, h, bits) == sv.SV_OK:
                    assert any("k_fill" in x for x in log()), nth     # the reset is still to be written
            sv.destroy_state(h)
        sv.batch_destroy(b)
    assert failed or "{api}" == ("hipLaunchKernel" if {graph} else "hipGraphLaunch")
    """))


@pytest.mark.parametrize("what", ["queued", "unusable", "permuted"])
def test_batch_refused_leaves_the_other_states(fake_hip, what):
    """A batch that is refused for one of its states leaves the others as they
    were: a reset that is not yet written stays to be written."""
    run(fake_hip, BATCH + textwrap.dedent(f"""
    hs, b = batch(True)
    if "{what}" == "queued":
        sv.apply_diag(hs[-1], [0], np.ones(2), "c64")
    elif "{what}" == "unusable":
        F.fake_fail(b"hipLaunchKernel", 1)
        assert code_of(sv.reduce_slices, hs[-1], np.arange(4, dtype=np.uint64)) == sv.SV_EDEVICE
    else:
        sv.permute_qubits(hs[-1], list(range(12))[::-1])
    for h in hs[:-1]:
        sv.reset(h)
    assert code_of(sv.batch_launch, b) == (sv.SV_ESTATE if "{what}" == "unusable" else sv.SV_EINVAL)
    for h in hs[:-1]:
        F.fake_clear()
        sv.reduce_slices(h, np.arange(4, dtype=np.uint64))
        assert any("k_fill" in x for x in log())
    """))


@pytest.mark.parametrize("nth", [1, 2, 3])
def test_noalloc_call_after_one_that_failed(fake_hip, nth):
    """The shared work array of reduce_slices_noalloc keeps nothing of a call
    that failed: it is idle when that call returns, and the next call, of
    another handle, starts with its ticket at zero."""
    run(fake_hip, f"""
    bits = np.arange(4, dtype=np.uint64)
    a, b = (sv.create_state(12, 0, "c64") for _ in range(2))
    for h in (a, b):
        sv.sync_state(h)
    F.fake_fail(b"hipMemcpyAsync", {nth})
    assert code_of(sv.reduce_slices_noalloc, a, bits) == sv.SV_EDEVICE
    assert F.fake_undone() == 0
    F.fake_clear()
    for _ in range(2):
        assert code_of(sv.reduce_slices_noalloc, b, bits) == sv.SV_OK
    assert "stale ticket" not in log()
    assert code_of(sv.reduce_slices, b, bits) == sv.SV_OK
    """)


@pytest.mark.parametrize("count", [0, 4, 1 << 12])
def test_reduction_without_pinned_memory(fake_hip, count):
    """No pinned memory to be had: a resident state's reduction copies."""
    run(fake_hip, f"""
    bits = np.arange({count}, dtype=np.uint64)
    h = sv.create_state(12, 0, "c64")
    F.fake_fail_always(b"hipHostMalloc", 1)
    for _ in range(2):
        assert code_of(sv.reduce_slices, h, bits) == sv.SV_OK
        assert code_of(sv.gather_amplitudes, h, bits) == sv.SV_OK
    F.fake_fail_always(b"hipHostMalloc", 0)
    F.fake_clear()
    assert code_of(sv.reduce_slices, h, bits) == sv.SV_OK
    assert not any(x.startswith("copy") for x in log())       # pinned again
    sv.destroy_state(h)
    assert F.fake_bad_frees() == 0
    """)


@pytest.mark.parametrize("left", [0, 1, 3])
def test_batch_with_few_streams(fake_hip, left):
    """A batch's graphs take as many streams as there are: each state's
    launches are in one of them, and the batch runs."""
    run(fake_hip, BATCH + textwrap.dedent(f"""
    hs, b = batch(True)
    F.fake_clear()
    sv.batch_launch(b)
    graphs = sum(x.startswith("graph") for x in log())
    assert graphs == 6
    hs = [sv.create_state(n, 0, "c64") for n in (20, 21, 22, 20, 23, 12)]
    for h in hs:
        sv.apply_fused(h, [1, 2, 3, 4, 5], unitary(5), "c64")
    F.fake_clear()
    F.fake_fail(b"hipStreamCreateWithFlags", 2 + {left})       # the batch's own comes first
    b = sv.batch_prepare(hs, graph=True)
    passes = [x for x in log() if x.startswith("launch") and ("k_split" in x or "k_stage" in x)]
    F.fake_clear()
    sv.batch_launch(b)
    assert sum(x.startswith("graph") for x in log()) == 1 + {left}
    assert len(passes) == 2 * 6                                # both variants, one pass a state
    sv.batch_destroy(b)
    """))


@pytest.mark.parametrize("where", ["resident", "whole", "slices", "pageable"])
def test_amplitude_bound_follows_reductions(fake_hip, where):
    """A reduction applies the queue, so the bound on the amplitudes, from
    which the split-fp16 passes take their scale, grows with it."""
    run(fake_hip, f"""
    n = {{"resident": 12, "whole": 12, "slices": 22, "pageable": 12}}["{where}"]
    tier = "{where}" != "resident"
    h = sv.create_state(n, 5 if tier else 0, "c64", tier=tier, pageable="{where}" == "pageable")
    sv.apply_diag(h, [1], np.array([1000.0, 1.0]), "c64")
    sv.reduce_slices(h, np.arange(4, dtype=np.uint64))
    sv.apply_diag(h, [1], np.array([1.0, 20.0]), "c64")
    sv.gather_amplitudes(h, np.arange(4, dtype=np.uint64))
    assert abs(sv.stage_forms(h)["amp_bound"] / 20000.0 - 1) < 1e-3
    sv.reset(h)
    assert sv.stage_forms(h)["amp_bound"] == 1.0
    """)


STAGED = """
def passes(h, n, dtype, widths, count):
    r = np.random.default_rng(n)
    for i in range(count):
        k = widths[i % len(widths)]
        sv.apply_fused(h, [int(q) for q in r.choice(min(n, 9), k, replace=False)], unitary(k, i), dtype)
    sv.sync_state(h)
"""


@pytest.mark.parametrize("limit", [160, 80])
def test_staged_kernels_get_their_lds(fake_hip, limit):
    """A staged kernel's LDS limit is set before its first launch, alone and in
    a captured batch, and not those of all the others; where the device gives
    a workgroup 80 KiB only, tiles stop at 13 positions and complex128 states
    take single sweeps."""
    run(fake_hip, STAGED + textwrap.dedent(f"""
    F.fake_lds_limit({limit} * 1024)
    for dtype in ("c64", "c128"):
        for n in (9, 12, 14, 16, 28):
            for stage in (9, 10, 12, 13, 14):
                for split in (1, 0):
                    h = sv.create_state(n, 0, dtype)
                    sv.set_option(h, sv.SV_OPT_STAGE, stage)
                    sv.set_option(h, sv.SV_OPT_SPLIT, split)
                    F.fake_clear()
                    for count in (1, 2, 5):
                        passes(h, n, dtype, (4, 5), count)
                        sv.reset(h)
                        passes(h, n, dtype, (5, 4), count)
                        sv.reduce_slices(h, np.arange(4, dtype=np.uint64))
                    lines = log()
                    assert not [x for x in lines if x.startswith("refused")], (dtype, n, stage, split)
                    assert sum(x.startswith("attribute") for x in lines) <= 24
                    staged = [x for x in lines if x.startswith("launch") and ("k_split" in x or "k_stage" in x)]
                    assert bool(staged) == (dtype == "c64" or {limit} == 160), (dtype, n, stage, split)
                    sv.destroy_state(h)
    for n in (12, 20, 23):
        h = sv.create_state(n, 0, "c64")
        for i, k in enumerate((5, 5, 4, 5)):
            sv.apply_fused(h, list(range(i, i + k)), unitary(k, i), "c64")
        F.fake_clear()
        b = sv.batch_prepare([h], graph=True)
        lines = log()
        capture = [i for i, x in enumerate(lines) if x.startswith("capture")]
        assert capture and not any(x.startswith("attribute") for x in lines[capture[0]:])
        assert not any(x.startswith("refused") for x in lines)
        sv.batch_launch(b)
        sv.batch_destroy(b)
    """))
