"""GPU checks of contraction deferral: sv_contract against the oracle's
contraction (App. A) on seeded random tensors, on the matrix-core path and
the plain path, complex64 and complex128; argument errors; and the whole
deferred pipeline (two tensors with EI / E2Q, contraction, the rest of the
circuit on the joint state) against the plain simulation."""
import numpy as np
import pytest

from oracle import deferral as D
from oracle import oracle as orc
from paper_1910_09534_amd import deferral, runner, sv
from paper_1910_09534_amd import workload as W

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _rand(size, rng):
    return (rng.standard_normal(size) + 1j * rng.standard_normal(size)) / np.sqrt(2)


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n1,n2,e,dtype", [
    (6, 7, 4, "c64"), (7, 8, 5, "c64"), (8, 7, 6, "c64"), (10, 9, 8, "c64"), (6, 10, 10, "c64"),
    (5, 7, 4, "c64"), (6, 6, 4, "c64"), (6, 7, 3, "c64"), (2, 3, 1, "c64"), (0, 0, 0, "c64"),
    (3, 2, 0, "c64"), (5, 6, 3, "c128"), (7, 8, 5, "c128")])
def test_contract_matches_oracle(n1, n2, e, dtype, fp32):
    """Matrix-core tiles (2^n2 >= 128, 2^n1 >= 64, 2^e >= 16; the split-fp16
    form, or the fp32 3M form with fp32) and the plain kernel (every other
    size) against the oracle, element by element."""
    torch = _torch()
    rng = np.random.default_rng(n1 * 1000 + n2 * 10 + e)
    t1 = _rand((1 << e) << n1, rng)
    t2 = _rand((1 << e) << n2, rng)
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    ndt = np.complex64 if dtype == "c64" else np.complex128
    g1 = torch.from_numpy(t1.astype(ndt)).cuda()
    g2 = torch.from_numpy(t2.astype(ndt)).cuda()
    out = torch.full((1 << (n1 + n2),), complex(7.0, 7.0), dtype=tdt, device="cuda")
    sv.contract(g1.data_ptr(), g2.data_ptr(), out.data_ptr(), n1, n2, e, dtype,
                torch.cuda.current_stream().cuda_stream, fp32=fp32)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.complex128)
    ref = D.contract_matrix(t1.astype(ndt), t2.astype(ndt), n1, n2, e)
    # FP32 sums over 2^e terms of unit-size products: error ~ 1e-7 sqrt(2^e)
    tol = 1e-12 if dtype == "c128" else 2e-6 * max(1.0, np.sqrt(1 << e))
    assert np.abs(got - ref).max() <= tol * max(1.0, np.abs(ref).max())
    assert orc.rel_l2(got, ref) <= (1e-13 if dtype == "c128" else 1e-5)


@pytest.mark.parametrize("n1,n2,e", [(4, 4, 2), (5, 4, 3), (4, 7, 4), (6, 5, 7), (5, 6, 9), (4, 4, 8), (4, 14, 8),
                                     (9, 11, 2), (5, 15, 5), (11, 11, 3)])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_contract_full_precision_tiles(n1, n2, e, dtype):
    """The matrix-core form in the data's own precision (complex128, and
    complex64 sizes outside the split form's): 16 x 16 outputs a wave with
    one and four steps at a time, the sum in one, 4 and 16 parts, and 32 x 32.
    The bound is that of a K-term sum of unit-size products, sqrt(K) eps
    with a factor 4 for the complex product's four real sums."""
    torch = _torch()
    rng = np.random.default_rng(n1 * 1000 + n2 * 10 + e + 7)
    ndt, eps = (np.complex64, 2.0 ** -24) if dtype == "c64" else (np.complex128, 2.0 ** -53)
    t1 = _rand((1 << e) << n1, rng).astype(ndt)
    t2 = _rand((1 << e) << n2, rng).astype(ndt)
    g1, g2 = torch.from_numpy(t1).cuda(), torch.from_numpy(t2).cuda()
    out = torch.full((1 << (n1 + n2),), complex(7.0, 7.0), dtype=g1.dtype, device="cuda")
    sv.contract(g1.data_ptr(), g2.data_ptr(), out.data_ptr(), n1, n2, e, dtype,
                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.complex128)
    ref = D.contract_matrix(t1, t2, n1, n2, e)
    bound = max(eps, 2.0 ** -52) * 4 * np.sqrt(1 << e)
    assert orc.rel_l2(got, ref) <= bound, orc.rel_l2(got, ref)


@pytest.mark.parametrize("n1,n2,e,fp32,scale", [
    (6, 7, 5, False, 1), (9, 9, 5, False, 1), (10, 10, 9, True, 1), (11, 11, 6, False, 1), (15, 5, 6, False, 1),
    (11, 11, 4, True, 1), (11, 11, 7, False, 1), (6, 15, 8, False, 1e10), (9, 10, 11, False, 1e-12),
    (7, 16, 4, False, 1), (13, 10, 5, False, 1e10), (16, 7, 6, False, 1e-12), (12, 14, 4, False, 1),
    (6, 20, 4, False, 1)])
def test_contract_tile_choice(n1, n2, e, fp32, scale):
    """Complex64 on both sides of each line of the tile choice: fp32 with the
    sum in one, 4 and 16 parts, the 3M form, split-fp16 tiles of 128 x 64 and
    128 x 128 outputs with one, two and more chunks, plain and non-temporal
    stores.  16 columns x2 are checked in full.  sqrt(K) eps for the sums with
    a factor 4 for the complex product's real sums, as above, and another 2
    for the 3M form's cancellations; the split adds at most 2^-21."""
    torch = _torch()
    rng = np.random.default_rng(n1 * 1000 + n2 * 10 + e + 11)
    t1 = (_rand((1 << e) << n1, rng) * scale).astype(np.complex64)
    t2 = _rand((1 << e) << n2, rng).astype(np.complex64)
    g1, g2 = torch.from_numpy(t1).cuda(), torch.from_numpy(t2).cuda()
    out = torch.full((1 << (n1 + n2),), complex(7.0, 7.0), dtype=g1.dtype, device="cuda")
    sv.contract(g1.data_ptr(), g2.data_ptr(), out.data_ptr(), n1, n2, e, "c64",
                torch.cuda.current_stream().cuda_stream, fp32=fp32)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([[0, (1 << n2) - 1], rng.integers(0, 1 << n2, 14)]))
    got = out.view(1 << n2, 1 << n1)[torch.from_numpy(rows).cuda()].cpu().numpy()
    ref = t2.reshape(1 << e, 1 << n2)[:, rows].T.astype(np.complex128) @ t1.reshape(1 << e, 1 << n1)
    assert orc.rel_l2(got.astype(np.complex128).ravel(), ref.ravel()) <= 8 * 2.0 ** -24 * np.sqrt(1 << e) + 2.0 ** -21
    assert np.abs(got - ref).max() <= 1e-5 * np.sqrt(1 << e) * scale


@pytest.mark.parametrize("n1,n2", [(4, 30), (30, 4)])
def test_contract_more_outputs_than_one_grid_dimension(n1, n2):
    """2^34 outputs with a side of 16: more work items than a grid dimension
    takes.  Stretches of outputs at both ends and in between are checked, the
    bound as above."""
    torch = _torch()
    e, big = 2, max(n1, n2)
    gen = torch.Generator(device="cuda").manual_seed(n1)
    t1 = torch.randn((1 << e) << n1, dtype=torch.complex64, device="cuda", generator=gen)
    t2 = torch.randn((1 << e) << n2, dtype=torch.complex64, device="cuda", generator=gen)
    out = torch.empty(1 << (n1 + n2), dtype=torch.complex64, device="cuda")
    sv.contract(t1.data_ptr(), t2.data_ptr(), out.data_ptr(), n1, n2, e, "c64",
                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    m1, m2, o = t1.view(1 << e, 1 << n1), t2.view(1 << e, 1 << n2), out.view(1 << n2, 1 << n1)
    width = 1 << 16
    try:
        for at in [0, 1 << 20, (1 << 29) - width // 2, (1 << big) - width] + [3 << k for k in range(17, 28)]:
            part = slice(at, at + width)
            if n2 == big:
                ref, got = m2[:, part].cpu().numpy().T.astype(np.complex128) @ m1.cpu().numpy(), o[part]
            else:
                ref, got = m2.cpu().numpy().T.astype(np.complex128) @ m1[:, part].cpu().numpy(), o[:, part]
            got = got.cpu().numpy().astype(np.complex128)
            assert orc.rel_l2(got.ravel(), ref.ravel()) <= 4 * 2.0 ** -24 * np.sqrt(1 << e), at
    finally:
        del t1, t2, out, m1, m2, o
        torch.cuda.empty_cache()


@pytest.mark.parametrize("s1,s2", [(1e-6, 1.0), (1.0, 3e5), (1e-15, 1e-12), (1e10, 1e-10)])
def test_contract_split_accuracy_independent_of_scale(s1, s2):
    """The split-fp16 form scales each tensor from its own largest component:
    tensors of very different sizes keep single-precision accuracy (no fp16
    overflow or underflow)."""
    torch = _torch()
    n1, n2, e = 7, 8, 6
    rng = np.random.default_rng(31)
    t1 = (_rand((1 << e) << n1, rng) * s1).astype(np.complex64)
    t2 = (_rand((1 << e) << n2, rng) * s2).astype(np.complex64)
    g1 = torch.from_numpy(t1).cuda()
    g2 = torch.from_numpy(t2).cuda()
    out = torch.zeros(1 << (n1 + n2), dtype=torch.complex64, device="cuda")
    sv.contract(g1.data_ptr(), g2.data_ptr(), out.data_ptr(), n1, n2, e, "c64",
                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.complex128)
    ref = D.contract_matrix(t1, t2, n1, n2, e)
    assert np.all(np.isfinite(got))
    assert orc.rel_l2(got, ref) <= 1e-5


def test_contract_rejects_bad_arguments():
    torch = _torch()
    a = torch.zeros(1 << 10, dtype=torch.complex64, device="cuda")
    b = torch.zeros(1 << 10, dtype=torch.complex64, device="cuda")
    o = torch.zeros(1 << 12, dtype=torch.complex64, device="cuda")
    with pytest.raises(sv.SVError):
        sv.contract(0, b.data_ptr(), o.data_ptr(), 6, 6, 4, "c64")
    with pytest.raises(sv.SVError):
        sv.contract(a.data_ptr() + 8, b.data_ptr(), o.data_ptr(), 6, 6, 4, "c64")     # misaligned
    with pytest.raises(sv.SVError):
        sv.contract(a.data_ptr(), b.data_ptr(), a.data_ptr(), 6, 6, 4, "c64")         # overlap
    with pytest.raises(sv.SVError):
        sv.contract(a.data_ptr(), b.data_ptr(), o.data_ptr(), 30, 20, 4, "c64")       # too large
    with pytest.raises(sv.SVError):
        sv.contract(a.data_ptr(), b.data_ptr(), o.data_ptr(), 6, 6, -1, "c64")
    with pytest.raises(sv.SVError):
        sv.contract(a.data_ptr(), b.data_ptr(), o.data_ptr(), 2, 2, 31, "c64")       # e above 30


@pytest.mark.parametrize("n,depth,ncycles", [(16, 8, 2), (16, 6, 4), (20, 8, 3)])
def test_deferred_pipeline_equals_simulation(n, depth, ncycles):
    """Two tensors (left and right halves of the grid) with EI / E2Q for the
    bridging gates of the first cycles, the contraction, then the rest of
    the circuit on the joint state: every amplitude equals the plain
    simulation."""
    _torch()
    c = W.sycamore_circuit(n, depth, seed=400 + n + ncycles)
    bits = np.arange(1 << n, dtype=np.uint64)
    res = runner.simulate_deferred(c, bits, deferral.grid_halves(n), ncycles)
    assert res["split"].n_bridging >= 2
    ref = orc.simulate(c)
    assert orc.rel_l2(res["amps"], ref) <= 1e-5
    assert abs(res["norm"] - 1.0) <= 1e-5
