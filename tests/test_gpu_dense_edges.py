"""The small eigensolver and the entropy at the sizes where their kernels change
form, against numpy and the oracle.

Eigenvalues to 1e-12 of the largest, vectors orthonormal to 1e-12 and with residual
1e-11 of the largest eigenvalue (the bars of test_gpu_kernels.py); entropies to 1e-10.
"""

import numpy as np
import pytest
import torch

from oracle import basis, observables
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
