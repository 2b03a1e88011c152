"""The CG paths behind mbl_pcg at the sizes where each can go wrong, against the
oracle's step-by-step PCG: one workgroup per column (sectors whose vector fits the
LDS: every rows-per-thread variant, its remainders, restarts between launches) and
panel-major vectors (sectors above: ragged panels, unaligned blocks, S^z != 0,
frozen guard columns, the largest chains).

Tolerances: m <= 9 CG steps amplify rounding by less than 1e4 (FP64 to 1e-9 of the
largest entry; FP32 to 2e-4 of the column norm).
"""

import time

import numpy as np
import pytest
import torch

from oracle import basis, hamiltonian, linalg, pcg as opcg
from paper_2012_00217_amd import workloads

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2012_00217_amd.api")
DEV = "cuda"


def _check(L, Sz, b, dtype, m, J=1.0, Delta=1.0, pad=0, offset=0):
    h = workloads.disorder(L, 4.0, 3)
    H = api.Hamiltonian(L, h, Sz=Sz, J=J, Delta=Delta)
    _, Ho = hamiltonian.sector_matrix(L, basis.nup_from_sz(L, Sz), J, Delta, h)
    sigma = 0.13
    R = workloads.random_block(H.n, b, seed=L + b)
    big = torch.zeros((H.n, b + pad), dtype=dtype, device=DEV)
    Rd = big[:, offset:offset + b]
    Rd.copy_(torch.from_numpy(R).to(DEV, dtype))
    W = H.pcg(Rd, sigma, m).double().cpu().numpy()
    Wr = opcg.pcg_fold(Ho, sigma, hamiltonian.fold_diagonal(Ho, sigma),
                       Rd.double().cpu().numpy(), m)
    if dtype == torch.float64:
        np.testing.assert_allclose(W, Wr, rtol=0, atol=1e-9 * max(1e-300, np.abs(Wr).max()))
    else:
        err = np.linalg.norm(W - Wr, axis=0)
        assert np.all(err <= 2e-4 * np.linalg.norm(Wr, axis=0))


# n = 2, 3, 10, 70, 924 (one row per thread), 1716 (2), 3432 (4), 5005 and 6435 (7),
# 8008 and 12870 (13); few up spins on a long chain (2024, 1)
@pytest.mark.parametrize("L,Sz", [(2, 0.0), (3, 0.5), (5, -0.5), (8, 0.0), (12, 0.0), (13, 0.5),
                                  (14, 0.0), (15, 1.5), (15, 0.5), (16, 2.0), (16, 0.0), (24, 9.0), (20, 10.0)])
@pytest.mark.parametrize("dtype,b,m", [(torch.float64, 1, 3), (torch.float64, 5, 1),
                                       (torch.float32, 3, 3), (torch.float32, 16, 0)])
def test_column_cg(L, Sz, dtype, b, m):
    _check(L, Sz, b, dtype, min(m, 2) if L < 5 else m)


@pytest.mark.parametrize("L,precision", [(12, "f64"), (13, "pcg32"), (14, "f64"), (15, "f64"),
                                         (16, "f64"), (16, "mixed")])
def test_column_cg_restarts_are_bitwise_one_launch(L, precision):
    """A solve with a time limit stops its CG every 32 steps to look at the clock
    and goes on from the saved state: the same bits as without."""
    h = workloads.disorder(L, 6.0, 1)
    H = api.Hamiltonian(L, h, Sz=0.5 * (L % 2))
    kw = dict(nev=4, block=8, tol=1e-8, precision=precision, pcg_iters=75, guard_cg=0.5, max_iter=3,
              raise_on_noconv=False)
    ev, V, rs, info = H.solve(0.1, **kw)
    ev2, V2, rs2, info2 = H.solve(0.1, max_seconds=600.0, **kw)
    assert np.array_equal(ev, ev2) and torch.equal(V, V2) and np.array_equal(rs, rs2)


# n = 12376 (L = 17, S^z = 3.5; a sector the column path takes), 19448, 18564,
# 24310, 48620; m = 9 replays a captured step
@pytest.mark.parametrize("L,Sz,J,Delta", [(17, 1.5, 0.7, -1.3), (18, 3.0, 1.0, 1.0),
                                          (17, -0.5, 1.0, 0.0), (18, 0.0, 1.3, 0.6)])
@pytest.mark.parametrize("dtype,b,m,pad,offset", [
    (torch.float64, 1, 9, 0, 0), (torch.float64, 2, 1, 0, 0), (torch.float64, 17, 3, 4, 1),
    (torch.float64, 34, 2, 2, 0), (torch.float32, 1, 3, 0, 0), (torch.float32, 3, 9, 5, 2),
    (torch.float32, 66, 3, 6, 4), (torch.float32, 64, 0, 0, 0)])
def test_panel_cg(L, Sz, J, Delta, dtype, b, m, pad, offset):
    _check(L, Sz, b, dtype, m, J, Delta, pad, offset)


@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_panel_cg_guard_columns(precision):
    """Columns beyond nev stop early, with nev not a whole number of panels."""
    L = 17
    h = workloads.disorder(L, 6.0, 2)
    H = api.Hamiltonian(L, h, Sz=0.5)
    _, Ho = hamiltonian.sector_matrix(L, basis.nup_from_sz(L, 0.5), 1.0, 1.0, h)
    ev, V, rs, info = H.solve(0.1, 5, 12, tol=1e-9, guard_cg=0.3, precision=precision)
    assert info["pcg_columns"] < 12 * info["pcg_steps"]
    assert linalg.residual_norms(Ho, ev, V.cpu().numpy()).max() <= 1e-9


@pytest.mark.parametrize("L,b,dtype", [(26, 6, torch.float32), (28, 3, torch.float64)])
def test_panel_cg_at_the_longest_chains(L, b, dtype, monkeypatch):
    """The panel CG against the row-major gather kernels (oracle-checked at full
    size elsewhere), which a launch schedule in the environment selects."""
    h = workloads.disorder(L, 4.0, 0)
    H = api.Hamiltonian(L, h)
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    R = torch.randn(H.n, b, dtype=dtype, device=DEV, generator=g)
    W = H.pcg(R, 0.2, 2)
    monkeypatch.setenv("MBL_APPLY_XCD_GROUP", "64")
    W0 = H.pcg(R, 0.2, 2)
    err = (W - W0).norm(dim=0) / W0.norm(dim=0)
    assert err.max().item() <= (1e-12 if dtype == torch.float64 else 2e-5)
    del W, W0, R
    torch.cuda.empty_cache()


@pytest.mark.parametrize("L,nup", [(24, 5), (20, 6)])
def test_sparse_sectors_keep_the_gather_kernels(L, nup, monkeypatch):
    """Far from half filling the blocks of rows are short: the same kernels as with a launch
    schedule asked for (here that of the default), to the bit."""
    H = api.Hamiltonian(L, workloads.disorder(L, 4.0, 1), Sz=nup - 0.5 * L)
    g = torch.Generator().manual_seed(5)
    R = torch.randn(H.n, 6, generator=g, dtype=torch.float64).to(DEV)
    W = H.pcg(R, 0.1, 5)
    monkeypatch.setenv("MBL_APPLY_LANE_BYTES", "64")
    assert torch.equal(W, H.pcg(R, 0.1, 5))


@pytest.mark.parametrize("max_seconds", [0.0, 600.0])
def test_column_cg_times_its_own_phases(max_seconds):
    """opts.timing with one workgroup per column: the two applies are timed each by
    itself inside the kernel, and the bytes are those of the columns that ran."""
    L, s = 14, 8
    H = api.Hamiltonian(L, workloads.disorder(L, 6.0, 1))
    t0 = time.perf_counter()
    ev, V, rs, info = H.solve(0.1, 4, 16, tol=1e-10, pcg_iters=75, guard_cg=0.4, max_iter=3,
                              raise_on_noconv=False, timing=True, max_seconds=max_seconds)
    wall = 1e3 * (time.perf_counter() - t0)
    steps, cols = info["pcg_steps"], info["pcg_columns"]
    assert cols < 16 * steps
    assert info["cg_launches_all"][0] == info["cg_apply1_launches"][0] == steps
    assert info["cg_apply1_bytes_all"][0] == pytest.approx(2 * H.n * s * cols + 12 * H.n * steps)
    assert info["cg_apply2_bytes_all"][0] == pytest.approx(6 * H.n * s * cols + 20 * H.n * steps)
    ms = [info["cg_apply1_ms_all"][0], info["cg_apply2_ms_all"][0]]
    assert ms[0] != ms[1] and min(ms) > 0.0
    # a gather of 3432 rows through one CU takes at least 0.1 us; both fit the solve
    assert min(ms) >= 1e-4 * cols / 16 and sum(ms) <= wall


@pytest.mark.parametrize("L,precision", [(12, "f64"), (13, "pcg32"), (14, "f64"), (15, "f64"),
                                         (16, "f64"), (16, "pcg32")])
def test_timing_the_column_cg_changes_no_bit(L, precision):
    H = api.Hamiltonian(L, workloads.disorder(L, 6.0, 1), Sz=0.5 * (L % 2))
    kw = dict(nev=4, block=8, tol=1e-8, precision=precision, pcg_iters=20, max_iter=2,
              raise_on_noconv=False)
    ev, V, rs, info = H.solve(0.1, **kw)
    ev2, V2, rs2, info2 = H.solve(0.1, timing=True, **kw)
    assert np.array_equal(ev, ev2) and torch.equal(V, V2) and np.array_equal(rs, rs2)


# 40 steps: at least 8 remain to be replayed.  Panels with 512 and 256 threads a tile (32
# tiles a panel; 129 panels), gather kernels as a schedule in the environment selects them
# and on a sector far from half filling, the two-pass kernels
@pytest.mark.parametrize("L,Sz,b,dtype,env", [
    (17, 0.5, 6, torch.float64, {}), (17, 0.5, 33, torch.float32, {}),
    (17, 0.5, 258, torch.float64, {}), (20, -4.0, 6, torch.float64, {}),
    (14, 0.0, 32, torch.float64, {"MBL_APPLY_LANE_BYTES": "64"}),
    (14, 0.0, 32, torch.float32, {"MBL_APPLY_LANE_BYTES": "64"}),
    (14, 0.0, 32, torch.float32, {"MBL_APPLY_SPLIT": "1"})])
def test_replayed_steps_are_bitwise_direct_launches(L, Sz, b, dtype, env, monkeypatch):
    """The captured step replayed against launches one by one, on the paths that replay;
    the caller's own work between the calls does not disturb it."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    H = api.Hamiltonian(L, workloads.disorder(L, 4.0, 2), Sz=Sz)
    R = torch.from_numpy(workloads.random_block(H.n, b, seed=11)).to(DEV, dtype)
    monkeypatch.setenv("MBL_PCG_GRAPH", "0")
    W_direct = H.pcg(R, 0.07, 40)
    assert torch.isfinite(W_direct).all() and W_direct.abs().max() > 0
    monkeypatch.setenv("MBL_PCG_GRAPH", "1")
    for _ in range(3):
        assert torch.equal(W_direct, H.pcg(R, 0.07, 40))
        (R * 2).sum().item()
