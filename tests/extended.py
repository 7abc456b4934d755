"""GMRES(3) smoothing steps (§5.3) in extended precision, and inputs whose residuals are smooth
(no test functions here)."""
import numpy as np

import oracle as O

LD = np.clongdouble


class Matrix:
    """A sparse matrix of the oracle applied in extended precision."""

    def __init__(self, A):
        A = A.tocsr()
        self.data, self.cols, self.rows = A.data.astype(LD), A.indices, A.indptr
        self.used = np.diff(A.indptr) > 0

    def __matmul__(self, x):
        y = np.zeros(len(self.used), LD)
        y[self.used] = np.add.reduceat(self.data * x[self.cols], self.rows[:-1][self.used])
        return y


def _dot(x, y):
    return (x.conj() * y).sum()


def gmres_step(A, u, f):
    """u after one GMRES(3) step on A u = f: Arnoldi with a second orthogonalisation, then the
    least-squares problem by Givens rotations."""
    r = f - A @ u
    z, H = [r / np.sqrt(_dot(r, r).real)], np.zeros((4, 3), LD)
    for j in range(3):
        w = A @ z[j]
        for _ in range(2):
            for i in range(j + 1):
                h = _dot(z[i], w)
                H[i, j] += h
                w = w - h * z[i]
        H[j + 1, j] = np.sqrt(_dot(w, w).real)
        z.append(w / H[j + 1, j])
    g = np.zeros(4, LD)
    g[0] = np.sqrt(_dot(r, r).real)
    for j in range(3):
        a, b = H[j, j], H[j + 1, j]
        rho = np.sqrt(abs(a) ** 2 + abs(b) ** 2)
        G = np.array([[a.conj(), b.conj()], [-b, a]]) / rho
        H[j:j + 2], g[j:j + 2] = G @ H[j:j + 2], G @ g[j:j + 2]
    for j in (2, 1, 0):
        g[j] = (g[j] - (H[j, j + 1:] * g[j + 1:3]).sum()) / H[j, j]
    return u + sum(g[j] * z[j] for j in range(3))


def cycle(H, u, f, pre, post):
    """u after one V(pre, post) cycle of the oracle's hierarchy H on A u = f."""
    A = [Matrix(a) for a in H.A]
    P, R = [Matrix(p) for p in H.P], [Matrix(r) for r in H.R]
    coarsest = H.A[-1].toarray()

    def level(l, u, f):
        if l == H.levels - 1:
            x = np.zeros_like(f)
            for _ in range(4):  # FP64 solves refined
                x = x + np.linalg.solve(coarsest, (f - A[l] @ x).astype(np.complex128))
            return x
        for _ in range(pre):
            u = gmres_step(A[l], u, f)
        fc = R[l] @ (f - A[l] @ u)
        u = u + P[l] @ level(l + 1, np.zeros_like(fc), fc)
        for _ in range(post):
            u = gmres_step(A[l], u, f)
        return u

    return level(0, u, f)


def amplification(A, f, u, shift):
    """sum |c_j| ||v_j|| / ||u|| for u = sum c_j v_j over v_j = (A - shift)^j f, j < 3: how far
    rounding of the v_j and c_j grows in u."""
    v = [f]
    for _ in range(2):
        v.append(A @ v[-1] - shift * v[-1])
    size = np.sqrt([_dot(x, x).real for x in v])
    q = [x / s for x, s in zip(v, size)]
    G = np.array([[_dot(a, b) for b in q] for a in q])
    c = np.array([_dot(a, u) for a in q])
    for k in range(3):
        for i in range(k + 1, 3):
            c[i] -= G[i, k] / G[k, k] * c[k]
            G[i] = G[i] - G[i, k] / G[k, k] * G[k]
    for k in (2, 1, 0):
        c[k] = (c[k] - (G[k, k + 1:] * c[k + 1:]).sum()) / G[k, k]
    return float(abs(c).sum() / np.sqrt(_dot(u, u).real))


def smooth_source(n, k=0.0, width=0.2):
    """W f of a Gaussian, times a plane wave of wavenumber k."""
    x = np.linspace(0.0, 1.0, n + 1)
    X, Y = np.meshgrid(x, x)
    f = np.exp(-((X - 0.45) ** 2 + (Y - 0.55) ** 2) / (2 * width ** 2)) * np.exp(1j * k * (0.8 * X + 0.6 * Y))
    return f * O.node_weights(n)


def distance(a, exact):
    """||a - exact|| / ||exact||"""
    d = np.asarray(a).ravel().astype(LD) - exact
    return float(np.sqrt(_dot(d, d).real / _dot(exact, exact).real))
