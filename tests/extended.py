"""Im Sigma^dec of a core state in long double, with a bound on what rounding may do.

The energies, grids and eta of `dyadic_system` are multiples of 2^-12 Ha, so
that every transition and every |eps_n - w| is exact in double and the error of
an FP64 evaluation is that of its arithmetic alone.  To first order a change
d(Pi) changes W = b^T [(1 - Pi)^-1 - 1] b by w^T d(Pi) w, w = (1 - Pi)^-1 b: with
every term of Pi off by a few eps,

    |dW| <= k eps (sum_ia |chi_ia| |(L^T w)_ia|^2 + |w - b|^2),

where the second sum stands for the solution's own rounding."""
import numpy as np

from workloads import system_from_config
from workloads.configs import small_config

LD, CLD = np.longdouble, np.clongdouble


def dyadic_system(n_occ=5, n_virt=35, n_aux=48, n_real=60, seed=9):
    s = system_from_config(small_config(n_occ=n_occ, n_virt=n_virt, n_aux=n_aux, n_core=1, n_real=n_real, seed=seed))
    s.eps = np.round(s.eps * 4096) / 4096
    s.eta = 1.0 / 256
    step = np.arange(n_real) - n_real + 1
    s.omega_real = (s.eps[0] + np.floor(step * (0.9 * 4096 / n_real)) / 4096)[None]
    return s


def _solve(A, b):
    A, b = A.copy(), b.copy()
    n = len(b)
    for k in range(n):
        m = A[k + 1:, k] / A[k, k]
        A[k + 1:, k + 1:] -= np.outer(m, A[k, k + 1:])
        b[k + 1:] -= m * b[k]
    for k in range(n - 1, -1, -1):
        b[k] = (b[k] - A[k, k + 1:] @ b[k + 1:]) / A[k, k]
    return b


def im_sigma_dec(s):
    """(value, bound / (k eps)) by grid point: the m = n term, weight -1 below eps_n
    and -1/2 at it."""
    no, N = s.n_occ, s.n_aux
    L = s.M_ov.reshape(N, -1).astype(LD)
    d = (s.eps[None, no:] - s.eps[:no, None]).ravel().astype(LD)
    b = s.M_oo[:, 0, 0].astype(LD)
    out, bound = [], []
    for w in s.omega_real[0]:
        x, f = s.eps[0] - w, (-1.0 if w < s.eps[0] else -0.5)
        z = CLD(complex(x, s.eta))
        chi = 4 * d / ((z - d) * (z + d))
        v = _solve(np.eye(N, dtype=LD) - (L * chi) @ L.T, b.astype(CLD))
        out.append(float(f * (b @ (v - b)).imag))
        g = L.T @ v
        bound.append(float(abs(f) * (np.sum(np.abs(chi) * np.abs(g) ** 2) + np.sum(np.abs(v - b) ** 2))))
    return np.array(out), np.array(bound)
