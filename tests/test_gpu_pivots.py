"""The register Gauss-Jordan's pivots where they matter: a strip whose first block is close to
singular.  Without PML a strip of constant medium is a real Dirichlet problem whose first block is
T_x + (2/h^2 - k^2) I; k^2 lies a relative distance d from 2/h^2 plus an eigenvalue of T_x.  The entries
of T_x are alike, so that candidates for a pivot differ little, and the solution inherits the error of
that block's inverse."""
import math

import numpy as np
import pytest
import scipy.sparse.linalg as spla

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.assemble import assemble_strip  # noqa: E402
from oracle.grid import geometry_from_workload  # noqa: E402

DEV = "cuda:0"
N, W_OUT, PAD = 60, 2, 5
WIDTH = N // 2 + W_OUT + 1 + PAD                     # columns of the first of two strips


def _problem(d):
    h = 1.0 / N
    lam = 2 / h ** 2 + 4 / h ** 2 * np.sin(np.arange(1, WIDTH + 1) * np.pi / (2 * (WIDTH + 1))) ** 2
    k2 = lam[np.argmin(abs(lam - (2 * math.pi / (10 * h)) ** 2))] * (1 + d)
    wl = W.Workload("first block", np.ones((N, N)), math.sqrt(k2), h, W_OUT, PAD, 2, [(5, 5)])
    wl.pml_s0 = wl.pml_iface_s0 = 0.0
    r = np.random.default_rng(1)
    shape = (2, N + 2 * W_OUT, WIDTH)
    return wl, r.standard_normal(shape) + 1j * r.standard_normal(shape)


def _exact(wl, f):
    """SuperLU with residuals and iterate in extended precision."""
    g = geometry_from_workload(wl)
    A = assemble_strip(g, g.strips[0]).tocsr()
    A.sort_indices()
    lu, data = spla.splu(A.tocsc(), permc_spec="COLAMD"), A.data.astype(np.clongdouble)
    out = []
    for r in f.reshape(len(f), -1).astype(np.clongdouble):
        x = np.zeros_like(r)
        for _ in range(5):
            x = x + lu.solve((r - np.add.reduceat(data * x[A.indices], A.indptr[:-1])).astype(np.complex128))
        out.append(x)
    return np.array(out).astype(np.complex128).reshape(f.shape)


# error: of an inversion that searches the whole column in full and divides; of one that compares 14
# bits of the squares and multiplies by reciprocals: 1.7e-8, 4.7e-7, 7.8e-1, 11
@pytest.mark.parametrize("d,error", [(1.3335e-4, 1.8e-9), (5.6234e-5, 1.0e-8), (1.7783e-6, 2.3e-2), (1.3335e-6, 3.3e-1)])
def test_strip_with_a_nearly_singular_first_block(d, error):
    from paper_1208_3956_amd import Helmholtz
    wl, f = _problem(d)
    H = Helmholtz(wl.c, wl.omega, wl.h, wl.J, wl.w_out, wl.w, pml_s0=0.0, pml_iface_s0=0.0, prec="c128", mode="full",
                  chunk=16, device=DEV).factor()
    assert H.strip_width[0] == WIDTH
    x = H.strip_solve(0, torch.from_numpy(f).to(DEV)).cpu().numpy()
    ref = _exact(wl, f)
    assert np.linalg.norm(x - ref) <= 3 * error * np.linalg.norm(ref)
    H.close()
