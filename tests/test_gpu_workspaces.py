"""Solves with blocks above 64 under an allocator that puts a guard band behind every
allocation: no kernel writes beyond the work space it was given, and the pairs are the
oracle's.

The eigensolver's work space is the one that depends on several sizes at once (one, two
and three blocks of columns share it), so the blocks lie on both sides of the sizes where
its kernels change form (192 columns in one workgroup).
"""

import threading

import numpy as np
import pytest
import torch

from oracle import hamiltonian, linalg, spectrum
from paper_2012_00217_amd import workloads

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2012_00217_amd.api")


class Guarded:
    """Allocator callbacks: each allocation is followed by BAND bytes of a known value,
    which are looked at when it is freed."""

    BAND = 10 << 20
    MARK = 0xA5

    def __init__(self):
        self.live, self.broken, self.frees = {}, [], 0
        self.lock = threading.Lock()

    def alloc(self, n, s):
        t = torch.empty(int(n) + self.BAND, dtype=torch.uint8, device="cuda")
        t[int(n):].fill_(self.MARK)
        torch.cuda.synchronize()
        with self.lock:
            self.live[t.data_ptr()] = (t, int(n))
        return t.data_ptr()

    def free(self, p, s):
        torch.cuda.synchronize()
        with self.lock:
            t, n = self.live.pop(p)
            self.frees += 1
        hit = (t[n:] != self.MARK).nonzero()
        if hit.numel():
            self.broken.append((n, int(hit[0]), int(hit[-1])))


@pytest.mark.parametrize("b,precision", [(64, "f64"), (65, "f64"), (96, "f64"), (96, "mixed"),
                                         (128, "f64"), (128, "pcg32")])
def test_solve_stays_inside_its_work_space(b, precision):
    L, nev = 12, 4
    h = workloads.disorder(L, 5.0, 3)
    _, Ho = hamiltonian.sector_matrix(L, L // 2, 1.0, 1.0, h)
    emin, emax = spectrum.bounds(Ho)
    sigma = spectrum.shift_from_density(emin, emax, 0.5)
    w_ref, _ = spectrum.nearest(Ho, sigma, nev)
    mem = Guarded()
    api.use_allocator(mem.alloc, mem.free)
    try:
        H = api.Hamiltonian(L, h)
        ev, V, rs, info = H.solve(sigma, nev, b, tol=1e-10, precision=precision)
        H.close()
    finally:
        api.use_torch_allocator()
    assert mem.frees > 0 and not mem.live
    assert mem.broken == []  # (bytes asked for, first and last byte written behind them)
    assert info["status"] == "MBL_OK"
    assert np.all(np.abs(ev - w_ref) <= 1e-10)
    assert np.all(linalg.residual_norms(Ho, ev, V.cpu().numpy()) <= 1e-10)
