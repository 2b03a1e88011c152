"""The small eigensolver and the entropy at the sizes where their kernels change
form, against numpy and the oracle.

Eigenvalues to 1e-12 of the largest, vectors orthonormal to 1e-12 and with residual
1e-11 of the largest eigenvalue (the bars of test_gpu_kernels.py); entropies to 1e-10.
"""

import numpy as np
import pytest
import torch

from oracle import basis, hamiltonian, linalg, observables, spectrum
from paper_2012_00217_amd import workloads

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2012_00217_amd.api")
DEV = "cuda"


# V in LDS to 48; full square in LDS to 136 (one block per thread to 86, two to 122,
# three above); packed triangle to 192; one launch per round above
@pytest.mark.parametrize("m", [2, 5, 47, 48, 49, 50, 85, 87, 88, 121, 123, 136, 137, 138, 191, 192,
                               193])
@pytest.mark.parametrize("kind", ["random", "graded", "degenerate", "diagonal"])
def test_small_eigh_forms(m, kind):
    rng = np.random.default_rng(m)
    if kind == "random":
        A = rng.standard_normal((m, m))
        A = A + A.T
    elif kind == "graded":  # positive definite, eigenvalues over 12 decades
        q, _ = np.linalg.qr(rng.standard_normal((m, m)))
        B = q * np.logspace(0, -6, m)[None, :]
        A = B.T @ B
    elif kind == "degenerate":  # equal diagonal entries: 45 degree rotations
        A = np.ones((m, m)) + 2.0 * np.eye(m)
    else:
        A = np.diag(np.arange(m, 0, -1.0))
    w, V = api.small_eigh(torch.from_numpy(A).to(DEV))
    w, V = w.cpu().numpy(), V.cpu().numpy()
    wr = np.linalg.eigvalsh(A)
    top = np.abs(wr).max()
    assert np.all(np.diff(w) >= 0)
    np.testing.assert_allclose(w, wr, rtol=0, atol=1e-12 * top)
    np.testing.assert_allclose(V.T @ V, np.eye(m), atol=1e-12)
    np.testing.assert_allclose(A @ V, V * w[None, :], atol=1e-11 * top)
    if kind == "graded":
        np.testing.assert_allclose(w, np.logspace(-12, 0, m), rtol=1e-6)


@pytest.mark.parametrize("scale", [1e-200, 1e-160, 1e150])
def test_small_eigh_extreme_scales(scale):
    """Squares of the entries would leave the range of a double."""
    rng = np.random.default_rng(1)
    for m in (8, 60, 150):
        A = rng.standard_normal((m, m))
        A = A + A.T
        w, V = api.small_eigh(torch.from_numpy(A * scale).to(DEV))
        np.testing.assert_allclose(w.cpu().numpy() / scale, np.linalg.eigvalsh(A), rtol=0,
                                   atol=1e-11 * m)
        np.testing.assert_allclose((V.T @ V).cpu().numpy(), np.eye(m), atol=1e-12)


@pytest.mark.parametrize("L,Sz,cut,nev", [(10, 0.0, 1, 3), (10, 0.0, 9, 1), (11, 1.5, 4, 17),
                                          (14, -3.0, 6, 2), (22, 0.0, 3, 50), (20, 0.0, 10, 2)])
def test_entropy_blocks(L, Sz, cut, nev):
    """Cuts at the ends, S^z != 0, more vectors than one chunk takes (L = 22), blocks
    above and below the size that is solved in one launch (L = 20)."""
    H = api.Hamiltonian(L, workloads.disorder(L, 2.0, 0), Sz=Sz)
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    V = torch.randn(H.n, nev + 3, dtype=torch.float64, device=DEV, generator=g)[:, 2:2 + nev]
    V = V / V.norm(dim=0)
    S = H.entanglement_entropy(V, cut)
    st = basis.enumerate_sector(L, basis.nup_from_sz(L, Sz))
    for j in sorted({0, 1, 42, 43, nev - 1}):
        if j < nev:
            want = observables.entanglement_entropy(V[:, j].cpu().numpy(), st, L, cut)
            assert abs(S[j] - want) <= 1e-10


def test_entropy_without_memory_for_a_copy_of_the_vectors():
    """The joint launches keep the vectors by columns; where the allocator has no room for
    that, each block is taken by itself."""
    L, nev = 12, 16
    H = api.Hamiltonian(L, workloads.disorder(L, 2.0, 0))
    V = torch.from_numpy(workloads.random_block(H.n, nev, seed=3)).to(DEV)
    V = V / V.norm(dim=0)
    want = H.entanglement_entropy(V)
    refused = []

    def alloc(n, s):
        if n > 128 << 10:
            refused.append(n)
            return 0
        return torch._C._cuda_cudaCachingAllocator_raw_alloc(int(n), int(s or 0))

    api.use_allocator(alloc, lambda p, s: torch._C._cuda_cudaCachingAllocator_raw_delete(int(p)))
    try:
        got = H.entanglement_entropy(V)
    finally:
        api.use_torch_allocator()
    assert refused
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-12)


def test_entropy_of_more_vectors_than_one_chunk_takes():
    """L = 22 cut at 6: every block is small, and the 256 MB of a chunk hold 47 vectors, so
    the last three come from a shorter second chunk."""
    L, cut, nev = 22, 6, 50
    H = api.Hamiltonian(L, workloads.disorder(L, 2.0, 0))
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    V = torch.randn(H.n, nev + 3, dtype=torch.float64, device=DEV, generator=g)[:, 2:2 + nev]
    V = V / V.norm(dim=0)
    S = H.entanglement_entropy(V, cut)
    st = basis.enumerate_sector(L, L // 2)
    for j in (0, 46, 47, 49):
        want = observables.entanglement_entropy(V[:, j].cpu().numpy(), st, L, cut)
        assert abs(S[j] - want) <= 1e-10


def _block(n, p, dtype, seed, lead=0):
    """n x p block of one-digit integers (every product and sum of a Gram is exact), rows
    `lead` elements further apart than p."""
    g = torch.Generator().manual_seed(seed)
    full = torch.randint(-3, 4, (n, p + lead), generator=g).to(dtype).to(DEV)
    return full[:, :p]


# tiles of 64 columns and quadrants of 32, 16-element folds, slabs of 32 rows, splits of
# 64 (FP64) and 256 (FP32) rows
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 257, 3432])
@pytest.mark.parametrize("p,q,lead", [(1, 1, 0), (17, 1, 0), (31, 33, 3), (64, 64, 0), (65, 16, 1),
                                      (130, 66, 2)])
def test_gram_edges(n, p, q, lead, dtype):
    A, B = _block(n, p, dtype, 1, lead), _block(n, q, dtype, 2, lead)
    a, b = A.double(), B.double()
    assert torch.equal(api.gram(A, B), (a.T @ b))
    C = api.gram(A, A)
    assert torch.equal(C, a.T @ a)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [33, 1000])
@pytest.mark.parametrize("p,q", [(3, 2), (17, 5), (64, 64), (67, 33)])
def test_gram_of_unaligned_columns(n, p, q, dtype):
    """Operands that begin one element into a row, one of them or both, up to the last
    element of their storage."""
    a, b = _block(n, p + 1, dtype, 1), _block(n, q + 1, dtype, 2)
    A, B = a[:, 1:], b[:, 1:]
    assert torch.equal(api.gram(A, B), A.double().T.contiguous() @ B.double())
    assert torch.equal(api.gram(A, b), A.double().T.contiguous() @ b.double())
    assert torch.equal(api.gram(A, A), A.double().T.contiguous() @ A.double())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("p", [15, 16, 31, 32, 33, 63, 64, 65, 96, 97, 192, 200])
def test_gram_of_one_operand_is_that_of_two(p, dtype):
    """Mirrored tiles and skipped quadrants against the full product, rounding and all."""
    g = torch.Generator().manual_seed(p)
    A = torch.randn(4097, p, generator=g, dtype=torch.float64).to(dtype).to(DEV)
    C = api.gram(A, A)
    assert torch.equal(C, C.T)
    # a product in FP64 has errors of the size that is looked for: 64-bit mantissas
    a = A.cpu().numpy().astype(np.longdouble)
    err = float(np.abs(C.cpu().numpy() - a.T @ a).max())
    # 4097 products of O(1) in the accumulation's type, summed over splits
    assert err <= 4097 * (2.3e-16 if dtype == torch.float64 else 1.2e-7) * 3


# tiles of 16 rows, 32 or 64 columns a wavefront, slabs of 8 (FP64) or 16 columns of A,
# groups of 32 or 64, chunks of C of 192 to 768; 32768 rows to the wide form
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [1, 15, 17, 130, 32767, 32768, 32785])
@pytest.mark.parametrize("p,q,lead", [(1, 1, 0), (3, 17, 1), (8, 32, 0), (33, 33, 3), (64, 64, 0),
                                      (97, 65, 2), (192, 64, 0), (193, 130, 1), (402, 34, 0),
                                      (840, 3, 4)])
def test_block_combine_edges(n, p, q, lead, dtype):
    A = _block(n, p, dtype, 3, lead)
    Cm = _block(p, q, torch.float64, 4)
    Y = api.block_combine(A, Cm)
    assert Y.dtype == dtype
    assert torch.equal(Y.double(), A.double() @ Cm)


# FP32 shapes by tiles of 16 rows (1024, 2048, 3072, 4096, 6144 of them) and blocks of 48 or
# 64 columns; rows of A at any alignment, up to the last element of their storage
@pytest.mark.parametrize("n", [16384, 16385, 32768, 32769, 49152, 49153, 65537, 98305])
@pytest.mark.parametrize("p,q", [(64, 64), (33, 33), (75, 41), (130, 65), (96, 96), (150, 96),
                                 (192, 64), (600, 48), (1030, 50)])
@pytest.mark.parametrize("offset", [0, 1])
def test_block_combine_fp32_shapes(n, p, q, offset):
    A = _block(n, p + offset, torch.float32, 3)[:, offset:]
    Cm = _block(p, q, torch.float64, 4)
    assert torch.equal(api.block_combine(A, Cm).double(), A.double() @ Cm)


@pytest.mark.parametrize("b", [33, 48, 64])
def test_orthonormalisation_in_place_of_fp32_blocks(b):
    """Mixed solves of a sector in each shape's range orthonormalise their FP32 blocks in
    place: the pairs are H's."""
    for L, Sz in ((17, 2.5), (17, 0.5), (18, 0.0)):
        H = api.Hamiltonian(L, workloads.disorder(L, 6.0, 1), Sz=Sz)
        ev, V, rs, info = H.solve(0.1, 4, b, tol=1e-9, precision="mixed", pcg_iters=120)
        _, Ho = hamiltonian.sector_matrix(L, basis.nup_from_sz(L, Sz), 1.0, 1.0,
                                          workloads.disorder(L, 6.0, 1))
        assert np.all(linalg.residual_norms(Ho, ev, V.cpu().numpy()) <= 1e-9)


def test_block_combine_keeps_non_finite_rows_apart():
    """Padding rows, columns and slabs take nothing from their neighbours."""
    A = torch.ones(40, 5, dtype=torch.float64, device=DEV)
    A[39, 0] = float("nan")
    A[7, 4] = float("inf")
    Y = api.block_combine(A, torch.ones(5, 3, dtype=torch.float64, device=DEV)).cpu()
    good = [r for r in range(40) if r not in (7, 39)]
    assert torch.equal(Y[good], torch.full((38, 3), 5.0, dtype=torch.float64))
    assert torch.isnan(Y[39]).all() and torch.isinf(Y[7]).all()


# Bases orthonormalised in place to 32 columns; Ritz coefficients in one workgroup's LDS
# to a block of 34; single and mixed blocks
@pytest.mark.parametrize("precision", ["f64", "mixed"])
@pytest.mark.parametrize("b", [5, 31, 32, 33, 34, 35, 48])
def test_solve_at_the_block_widths_where_kernels_change(b, precision):
    L, nev = 10, 4
    h = workloads.disorder(L, 5.0, 3)
    _, Ho = hamiltonian.sector_matrix(L, L // 2, 1.0, 1.0, h)
    emin, emax = spectrum.bounds(Ho)
    sigma = spectrum.shift_from_density(emin, emax, 0.45)
    w_ref, _ = spectrum.nearest(Ho, sigma, nev)
    H = api.Hamiltonian(L, h)
    ev, V, rs, info = H.solve(sigma, nev, b, tol=1e-10, precision=precision)
    assert info["status"] == "MBL_OK"
    assert np.all(np.abs(ev - w_ref) <= 1e-10)
    assert np.all(linalg.residual_norms(Ho, ev, V.cpu().numpy()) <= 1e-10)
    lo, hi = H.spectrum_bounds(1e-9)[:2]
    assert abs(lo - emin) <= 1e-8 and abs(hi - emax) <= 1e-8


def test_block_combine_under_graph_capture():
    """The wide form with more than 64 KB of LDS (C of 192 x 64 in FP64)."""
    A, Cm = _block(32800, 192, torch.float64, 5), _block(192, 64, torch.float64, 6)
    ref = api.block_combine(A, Cm)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = api.block_combine(A, Cm)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
