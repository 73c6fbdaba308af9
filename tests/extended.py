"""Strip solves, sweeps and reduced operator in extended precision: the oracle's matrices, SuperLU with
residuals and iterates in long double."""
import numpy as np

from oracle.assemble import assemble_global, assemble_strip
from oracle.dd import StripSolvers

LD = np.clongdouble


class Matrix:
    def __init__(self, A):
        A = A.tocsr()
        A.sort_indices()
        self.cols, self.start, self.data = A.indices, A.indptr[:-1], A.data.astype(LD)

    def __matmul__(self, x):
        return np.add.reduceat(self.data * x[self.cols], self.start)


class Sweeps(StripSolvers):
    def __init__(self, g):
        super().__init__(g)
        self.A = Matrix(assemble_global(g))
        self.strip = [Matrix(assemble_strip(g, st)) for st in g.strips]

    def solve(self, s, rhs):
        r, x = rhs.ravel().astype(LD), np.zeros(rhs.size, LD)
        for _ in range(5):
            x = x + self.lu[s].solve((r - self.strip[s] @ x).astype(np.complex128))
        return x.reshape(rhs.shape)

    def P(self, f):
        """P f = v + w as in oracle.dd.sweep."""
        g = self.g
        ih2 = 1 / np.longdouble(g.h) ** 2
        v, w = np.zeros(f.shape, LD), np.zeros(f.shape, LD)
        prev = None
        for s, st in enumerate(g.strips):
            rhs, (lo, hi) = np.zeros(g.strip_shape(st), LD), st.core
            rhs[..., lo - st.a:hi - st.a] = f[..., lo:hi]
            if prev is not None:
                b, (q, x) = g.beta[s], prev
                d = (x[..., b - q.a] - x[..., b - 1 - q.a]) * ih2
                rhs[..., b - 1 - st.a] -= d
                rhs[..., b - st.a] -= d
            x = self.solve(s, rhs)
            v[..., lo:hi] = x[..., lo - st.a:hi - st.a]
            prev = (st, x)
        res, prev = f - (self.A @ v.ravel()).reshape(f.shape), None
        for s in range(g.J - 1, -1, -1):
            st = g.strips[s]
            rhs, (lo, hi) = np.zeros(g.strip_shape(st), LD), st.keep_dn
            rhs[..., lo - st.a:hi - st.a] = res[..., lo:hi]
            if prev is not None:
                b, (q, x) = g.beta[s + 1], prev
                d = (x[..., b + 1 - q.a] - x[..., b - q.a]) * ih2
                rhs[..., b - st.a] += d
                rhs[..., b + 1 - st.a] += d
            x = self.solve(s, rhs)
            w[..., lo:hi] = x[..., lo - st.a:hi - st.a]
            prev = (st, x)
        return v + w

    def AP_reduced(self, psi):
        g = self.g
        cols, f = g.reduced_columns(), np.zeros(g.field_shape, LD)
        f[..., cols] = psi
        return (self.A @ self.P(f).ravel()).reshape(f.shape)[..., cols].astype(np.complex128)
