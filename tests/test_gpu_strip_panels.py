"""Strip solves at the panel widths and chunk sizes where the strip solver's kernels change
form: 1, 2, 3, 4 right-hand sides (the matrix-vector chains; 3 runs in a panel of 4), 5 and
16 (one group of the matrix-core form, ragged and full) and 17 (two groups), over chunks
of one and two interior rows (no backward step, one), an even and an odd number of them, and
a single chunk, against the oracle's SuperLU strip solves."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.dd import StripSolvers  # noqa: E402
from oracle.grid import geometry_from_workload  # noqa: E402

DEV = "cuda:0"
TOL = {"c128": 1e-10, "mixed": 2e-4}     # the strip-solve bars of the parity tests


@pytest.fixture(scope="module")
def case():
    c = 1.0 + 0.4 * np.random.default_rng(41).random((30, 30))
    wl = W.small(n=30, J=3, w_out=6, w=5, c=c, nsrc=1, seed=42)
    g = geometry_from_workload(wl)
    return wl, g, StripSolvers(g)


@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("chunk", [2, 3, 10, 11, 64])
def test_strip_solve_panel_widths(case, prec, chunk):
    from paper_1208_3956_amd import Helmholtz
    wl, g, S = case
    H = Helmholtz(wl.c, wl.omega, wl.h, wl.J, wl.w_out, wl.w, prec=prec, chunk=chunk, device=DEV).factor()
    for nrhs in (1, 2, 3, 4, 5, 16, 17):
        rng = np.random.default_rng(100 * chunk + nrhs)
        for s, st in enumerate(g.strips):
            r = rng.standard_normal((nrhs, g.N_y, st.W)) + 1j * rng.standard_normal((nrhs, g.N_y, st.W))
            x = H.strip_solve(s, torch.from_numpy(r).to(DEV)).cpu().numpy()
            for k in range(nrhs):
                ref = S.solve(s, r[k])
                err = np.linalg.norm(x[k] - ref) / np.linalg.norm(ref)
                worst = np.abs(x[k] - ref).max() / np.abs(ref).max()
                assert err < TOL[prec] and worst < TOL[prec], (nrhs, s, k, err, worst)
    H.close()
