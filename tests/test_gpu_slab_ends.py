"""Slab factorisations and solves from both ends of y to a middle plane, at the numbers of
planes where the ends differ: the fewest (4 and 5 planes, an upper end of one), an even and
an odd number of them; one right-hand side, a full group of 16 and one more, both precisions,
against the oracle's SuperLU slab solves."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.dd import StripSolvers  # noqa: E402
from oracle.grid import geometry_from_workload  # noqa: E402

DEV = "cuda:0"
TOL = {"c128": 1e-10, "mixed": 2e-4}     # the slab-solve bars of the 3-D parity tests


@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("ny,w_out", [(2, 1), (3, 1), (5, 3), (8, 3)])
def test_slab_solve_from_both_ends(prec, ny, w_out):
    from paper_1208_3956_amd import Helmholtz
    c = 1.0 + 0.4 * np.random.default_rng(ny).random((9, ny, 12))
    wl = W.small3(n=12, J=2, w_out=w_out, w=3, c=np.ones((12, 12, 12)), nsrc=1).with_(c=c)
    g = geometry_from_workload(wl)
    S = StripSolvers(g)
    H = Helmholtz(wl.c, wl.omega, wl.h, wl.J, wl.w_out, wl.w, prec=prec, device=DEV).factor()
    assert H.N_y == ny + 2 * w_out
    for nrhs in (1, 16, 17):
        rng = np.random.default_rng(nrhs)
        for s, st in enumerate(g.strips):
            shape = (nrhs, H.N_z, H.N_y, st.W)
            r = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
            x = H.strip_solve(s, torch.from_numpy(r).to(DEV)).cpu().numpy()
            for k in range(nrhs):
                ref = S.solve(s, r[k])
                err = np.linalg.norm(x[k] - ref) / np.linalg.norm(ref)
                worst = np.abs(x[k] - ref).max() / np.abs(ref).max()
                assert err < TOL[prec] and worst < TOL[prec], (nrhs, s, k, err, worst)
    H.close()


# W N_z unknowns a plane: one block of 64 or of 128 columns, 128 and 64, two of 128
@pytest.mark.parametrize("nz,Bp", [(2, 64), (8, 128), (12, 192), (17, 256)])
def test_slab_solve_by_column_blocks(nz, Bp):
    """Complex64 elimination of a plane in blocks of 128 columns and a last one of 64, each
    diagonal block updated by its own workgroup."""
    from paper_1208_3956_amd import Helmholtz
    c = 1.0 + 0.4 * np.random.default_rng(nz).random((nz, 4, 12))
    wl = W.small3(n=12, J=2, w_out=1, w=3, c=np.ones((12, 12, 12)), nsrc=1).with_(c=c)
    g = geometry_from_workload(wl)
    S = StripSolvers(g)
    H = Helmholtz(wl.c, wl.omega, wl.h, wl.J, wl.w_out, wl.w, prec="mixed", device=DEV).factor()
    assert max(st.W for st in g.strips) * H.N_z in range(Bp - 63, Bp + 1)
    rng = np.random.default_rng(Bp)
    for s, st in enumerate(g.strips):
        shape = (2, H.N_z, H.N_y, st.W)
        r = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
        x = H.strip_solve(s, torch.from_numpy(r).to(DEV)).cpu().numpy()
        for k in range(2):
            ref = S.solve(s, r[k])
            err = np.linalg.norm(x[k] - ref) / np.linalg.norm(ref)
            assert err < TOL["mixed"], (s, k, err)
    H.close()
