"""The dense strip operators near a resonance: without PML a strip of constant medium is a real Dirichlet
problem, and with k^2 a relative distance d from an eigenvalue of a box of its first R rows the block
that completes the box is as ill-conditioned as 1/d.  Where that is a separator eliminated in a join of
chunks the handle goes over to the block substitutions; where no join meets it the dense operator is as
accurate as they are.  Against extended precision."""
import math

import numpy as np
import pytest

import workloads as W
from extended import Sweeps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.grid import geometry_from_workload  # noqa: E402

DEV = "cuda:0"
NY, NX, W_OUT, PAD = 158, 60, 2, 5
WIDTH = NX // 2 + W_OUT + 1 + PAD


def _problem(rows, d):
    h = 1.0 / NY
    a, b = (4 / h ** 2 * np.sin(np.arange(1, n + 1) * np.pi / (2 * (n + 1))) ** 2 for n in (WIDTH, rows))
    lam = (a[:, None] + b[None]).ravel()
    k2 = lam[np.argmin(abs(lam - (2 * math.pi / (10 * h)) ** 2))] * (1 + d)
    wl = W.Workload("box", np.ones((NY, NX)), math.sqrt(k2), h, W_OUT, PAD, 2, [(5, 5)])
    wl.pml_s0 = wl.pml_iface_s0 = 0.0
    r = np.random.default_rng(rows)
    shape = (2, NY + 2 * W_OUT, 2)
    return wl, r.standard_normal(shape) + 1j * r.standard_normal(shape)


def _reduced(wl, psi, prec, chunk, **kw):
    from paper_1208_3956_amd import Helmholtz
    H = Helmholtz(wl.c, wl.omega, wl.h, wl.J, wl.w_out, wl.w, pml_s0=0.0, pml_iface_s0=0.0, prec=prec, chunk=chunk,
                  device=DEV, **kw).factor()
    assert H.strip_width[0] == WIDTH
    H.set_kernel_timing(True)
    out = H.apply_AP_reduced(torch.from_numpy(psi).to(DEV)).cpu().numpy()
    dense = H.kernel_times()["phase_a"][0] == 0      # no block substitution ran
    H.close()
    return out, dense


# chunks of 8 rows are joined (boxes of 7, 31 rows are eliminated on the way), chunks of 48 are not.
# condition estimates: 3.5e3, 3.7e7, 3.7e9; 3.6e6
@pytest.mark.parametrize("chunk,rows,d,dense", [
    (8, 31, 1e-2, {"c128": True, "mixed": True}), (8, 31, 1e-6, {"c128": False, "mixed": True}),
    (8, 31, 1e-8, {"c128": False, "mixed": False}), (8, 7, 1e-6, {"c128": False, "mixed": True}),
    (48, 47, 1e-4, {"c128": True, "mixed": True}), (48, 47, 1e-6, {"c128": True, "mixed": True}),
    (48, 20, 1e-6, {"c128": True, "mixed": True})])
def test_reduced_operator_near_a_resonance(chunk, rows, d, dense):
    wl, psi = _problem(rows, d)
    S = Sweeps(geometry_from_workload(wl))
    ref = np.array([S.AP_reduced(p) for p in psi])
    for prec in ("c128", "mixed"):
        out, is_dense = _reduced(wl, psi, prec, chunk, mode="reduced")
        blocks, none = _reduced(wl, psi, prec, chunk, mode="full", batch_fuse=True)
        err, own = (np.linalg.norm(x - ref) / np.linalg.norm(ref) for x in (out, blocks))
        print(prec, f"error {err:.2e}, of the block substitutions {own:.2e}", flush=True)
        assert is_dense == dense[prec] and not none
        # rounding of another order of the same products: within an order of magnitude (or 1e-10,
        # the bar of the preconditioner's parity)
        assert err <= max(10 * own, 1e-10), (prec, err, own)
