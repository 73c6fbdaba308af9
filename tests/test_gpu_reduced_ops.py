"""The dense strip operators of the reduced form at the sizes where their layout changes: one
chunk (no separators) and several, chunks whose rows are and are not a multiple of the
16-row tiles, a ragged last chunk, one joining level to many, and a chunk size above which
they are not built; two strips and more; panels of one, one full, one and a ragged, and three
groups of 16 right-hand sides.  Reduced A P against the oracle on the first and last
right-hand side, and against a full-form handle that fuses its strip solves (it runs the block
substitutions) on every right-hand side.  A panel of one right-hand side after a wider one
holding infinities must not see them."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.assemble import assemble_global  # noqa: E402
from oracle.dd import StripSolvers, apply_AP_reduced, apply_P, to_reduced  # noqa: E402
from oracle.grid import geometry_from_workload  # noqa: E402

DEV = "cuda:0"
TOL = {"c128": 1e-10, "mixed": 2e-4}     # the preconditioner bars of the parity tests


def _case(n, J):
    c = 1.0 + 0.4 * np.random.default_rng(n).random((n, n))
    wl = W.small(n=n, J=J, w_out=6, w=5, c=c, nsrc=1, seed=n + 1)
    g = geometry_from_workload(wl)
    return wl, g, assemble_global(g), StripSolvers(g)


@pytest.fixture(scope="module")
def cases():
    return {(n, J): _case(n, J) for n, J in ((30, 2), (150, 5))}


def _handle(wl, prec, mode, chunk, **kw):
    from paper_1208_3956_amd import Helmholtz
    return Helmholtz(wl.c, wl.omega, wl.h, wl.J, wl.w_out, wl.w, prec=prec, mode=mode, chunk=chunk, **kw,
                     device=DEV).factor()


# padded rows 42 and 162; chunks joined to 42 (one chunk), 128 / 64, 72, 96 / 48, 80 rows; 130: not joined
@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("n,J,chunk", [(30, 2, 2), (30, 2, 9), (150, 5, 2), (150, 5, 9), (150, 5, 16), (150, 5, 40),
                                       (150, 5, 48), (150, 5, 130)])
def test_reduced_operator(cases, prec, n, J, chunk):
    wl, g, A, S = cases[(n, J)]
    H, B = _handle(wl, prec, "reduced", chunk), _handle(wl, prec, "full", chunk, batch_fuse=True)
    for nrhs in (1, 16, 17, 33):
        rng = np.random.default_rng(10 * chunk + nrhs)
        shape = (nrhs, g.N_y, 2 * (g.J - 1))
        psi = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
        t = torch.from_numpy(psi).to(DEV)
        out = H.apply_AP_reduced(t).cpu().numpy()
        other = B.apply_AP_reduced(t).cpu().numpy()
        for k in range(nrhs):
            ref = apply_AP_reduced(g, S, A, psi[k]) if k in (0, nrhs - 1) else other[k]
            err = np.linalg.norm(out[k] - ref) / np.linalg.norm(ref)
            worst = np.abs(out[k] - ref).max() / np.abs(ref).max()
            assert err < TOL[prec] and worst < TOL[prec], (nrhs, k, err, worst)
    H.close()
    B.close()


@pytest.mark.parametrize("prec", ["c128", "mixed"])
def test_reduced_operator_keeps_right_hand_sides_apart(cases, prec):
    wl, g, A, S = cases[(150, 5)]
    H = _handle(wl, prec, "reduced", 16)
    rng = np.random.default_rng(3)
    shape = (19, g.N_y, 2 * (g.J - 1))
    psi = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to(DEV)
    one = H.apply_AP_reduced(psi[:1])
    bad = psi.clone()
    bad[1:] = complex(float("inf"), 0.0)
    assert torch.equal(H.apply_AP_reduced(bad)[0], one[0])
    assert torch.equal(H.apply_AP_reduced(psi[:1])[0], one[0])
    assert torch.equal(H.apply_AP_reduced(psi)[0], one[0])
    H.close()


# panels of up to four, of up to 16 (tiles of four right-hand sides in FP64) and of several groups:
# sums over fewer than 1000 products of FP64 (FP32) in any order
@pytest.mark.parametrize("prec,tol", [("c128", 1e-12), ("mixed", 5e-4)])
@pytest.mark.parametrize("n,J,chunk", [(30, 2, 9), (150, 5, 2), (150, 5, 9)])
def test_reduced_operator_few_right_hand_sides(cases, prec, tol, n, J, chunk):
    wl, g, A, S = cases[(n, J)]
    H = _handle(wl, prec, "reduced", chunk)
    rng = np.random.default_rng(chunk)
    shape = (49, g.N_y, 2 * (g.J - 1))
    psi = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to(DEV)
    wide = H.apply_AP_reduced(psi)
    for nrhs in (1, 2, 3, 4, 5, 8, 9, 13, 16, 17, 32):
        got = H.apply_AP_reduced(psi[:nrhs].clone())
        assert (got - wide[:nrhs]).abs().max() <= tol * wide.abs().max(), nrhs
    H.close()


# chunks of the strip solver: many (two-level separators), four (one separator chain), two, one
@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("mode", ["full", "reduced"])
@pytest.mark.parametrize("n,J,chunk", [(30, 2, 9), (150, 5, 9), (150, 5, 45), (150, 5, 96), (30, 2, 64)])
def test_P_from_batches_of_strips(cases, prec, mode, n, J, chunk):
    """P f and the restart's right-hand side: every strip's own source, the sweeps' inputs
    and the fields in batches of strips, for panels of each strip-solver form."""
    wl, g, A, S = cases[(n, J)]
    H = _handle(wl, prec, mode, chunk)
    rng = np.random.default_rng(chunk)
    f = rng.standard_normal((17, g.N_y, g.N_x)) + 1j * rng.standard_normal((17, g.N_y, g.N_x))
    ref = [apply_P(g, S, A, f[k]) for k in (0, 1, 2, 4, 16)]
    bref = [to_reduced(g, f[k] - (A @ p.ravel()).reshape(p.shape)) for k, p in zip((0, 1, 2, 4, 16), ref)]
    for nrhs in (1, 2, 3, 5, 17):
        t = torch.from_numpy(f[:nrhs]).to(DEV)
        out = H.apply_P(t).cpu().numpy()
        b = H.restart_rhs_reduced(t).cpu().numpy()
        for k, r, br in zip((0, 1, 2, 4, 16), ref, bref):
            if k >= nrhs:
                continue
            err = np.linalg.norm(out[k] - r) / np.linalg.norm(r)
            worst = np.abs(out[k] - r).max() / np.abs(r).max()
            assert err < TOL[prec] and worst < TOL[prec], (nrhs, k, err, worst)
            # the stencil amplifies what P leaves, as in the parity test of this entry point
            err = np.linalg.norm(b[k] - br) / np.linalg.norm(br)
            assert err < {"c128": 1e-9, "mixed": 1e-3}[prec], (nrhs, k, err)
    H.close()
