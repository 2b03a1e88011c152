"""The block apply by tiles of rows against the gather kernels, to the bit, and the oracle.

Both add the bonds of a row in the same order and end in the same fused multiply-add, so
every block must come out the same: ragged and unaligned widths (pieces that overlap),
slices that overlap, widths below one 16-byte piece, padded rows, odd chains, S^z != 0,
short chains and both sides of the limits of the path.
"""

import numpy as np
import pytest
import torch

from oracle import basis, hamiltonian
from paper_2012_00217_amd import workloads

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2012_00217_amd.api")
DEV = "cuda"


def _both(monkeypatch, H, X, sigma, out=None):
    Y = H.apply(X, sigma, out=out).clone()
    monkeypatch.setenv("MBL_APPLY_SLOTS_PER_XCD", "256")
    Z = H.apply(X, sigma)
    monkeypatch.delenv("MBL_APPLY_SLOTS_PER_XCD")
    return Y, Z


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L,Sz", [(11, 0.5), (12, 0.0), (13, -0.5), (14, 2.0), (16, 0.0),
                                  (17, 0.5), (20, 0.0), (20, -3.0), (20, 4.0), (21, 2.5)])
@pytest.mark.parametrize("b,pad,offset", [(1, 0, 0), (2, 1, 1), (3, 0, 0), (4, 0, 0), (5, 2, 1),
                                          (17, 0, 0), (18, 3, 2), (19, 0, 0), (36, 4, 1),
                                          (37, 0, 0), (64, 0, 0), (73, 1, 0)])
def test_tiles_equal_the_gather(monkeypatch, L, Sz, b, pad, offset, dtype):
    H = api.Hamiltonian(L, workloads.disorder(L, 4.0, 2), Sz=Sz, Delta=0.7)
    g = torch.Generator(device=DEV).manual_seed(L * 100 + b)
    big = torch.randn(H.n, b + pad, generator=g, dtype=dtype, device=DEV)
    X = big[:, offset:offset + b] if offset + b <= b + pad else big[:, :b]
    Y, Z = _both(monkeypatch, H, X, 0.3)
    assert torch.equal(Y, Z)


# one slice to 208 bytes, then several; whole lines (with a stride or an offset that breaks
# them); few tiles, whose slices are halved
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("L", [14, 18, 19, 20])
@pytest.mark.parametrize("row,pad,offset", [(192, 0, 0), (208, 0, 0), (216, 0, 0), (320, 0, 0),
                                            (400, 8, 8), (624, 0, 0), (632, 0, 0), (800, 0, 0),
                                            (1152, 0, 0), (1152, 128, 0), (1152, 128, 32),
                                            (1152, 24, 0), (2048, 0, 0), (2040, 8, 8)])
def test_slices_equal_the_gather(monkeypatch, L, row, pad, offset, dtype):
    es = torch.finfo(dtype).bits // 8
    H = api.Hamiltonian(L, workloads.disorder(L, 4.0, 2), Sz=0.5 * (L % 2), Delta=0.7)
    g = torch.Generator(device=DEV).manual_seed(L * 100 + row)
    big = torch.randn(H.n, (row + pad) // es, generator=g, dtype=dtype, device=DEV)
    Y, Z = _both(monkeypatch, H, big[:, offset // es:(offset + row) // es], 0.3)
    assert torch.equal(Y, Z)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_tiles_write_their_columns_only(monkeypatch, dtype):
    L, b = 16, 19
    H = api.Hamiltonian(L, workloads.disorder(L, 4.0, 2))
    X = torch.randn(H.n, b, dtype=dtype, device=DEV)
    out = torch.full((H.n, b + 6), -7.0, dtype=dtype, device=DEV)
    Y, Z = _both(monkeypatch, H, X, 0.3, out=out[:, 3:3 + b])
    assert torch.equal(Y, Z)
    assert (out[:, :3] == -7).all() and (out[:, 3 + b:] == -7).all()


@pytest.mark.parametrize("L,Sz", [(12, 0.0), (13, 0.5), (15, -0.5)])
def test_tiles_against_the_oracle(L, Sz):
    h = workloads.disorder(L, 4.0, 3)
    H = api.Hamiltonian(L, h, Sz=Sz, J=1.3, Delta=0.6)
    _, Ho = hamiltonian.sector_matrix(L, basis.nup_from_sz(L, Sz), 1.3, 0.6, h)
    X = workloads.random_block(H.n, 7, seed=1)
    Y = H.apply(torch.as_tensor(np.asarray(X), dtype=torch.float64).to(DEV), 0.2).cpu().numpy()
    ref = Ho @ X - 0.2 * X
    np.testing.assert_allclose(Y, ref, rtol=0, atol=1e-12 * np.abs(ref).max())


def test_tiles_under_graph_capture():
    H = api.Hamiltonian(16, workloads.disorder(16, 4.0, 2))
    X = torch.randn(H.n, 24, dtype=torch.float64, device=DEV)
    out = torch.empty_like(X)
    ref = H.apply(X, 0.1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        H.apply(X, 0.1, out=out)
    for _ in range(3):
        X.mul_(1.0)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
