"""The FMM of one order p on the oracle's tree and lists, in numpy: the harmonic
field at points inside the leaves, its derivative, and the logarithmic potential at
the sources, so that results can be compared at the same truncation.  Expansions
scaled by the box radius r (all boxes must have an extent):

    multipole   a_k = sum_j m_j ((z_j - c) / r)^k                     k < p
    local       phi(z) = sum_l b_l ((z - c) / r)^l                    l < p
    M2M  a^P_k = sum_l C(k, l) rho^l tau^(k-l) a^C_l
    M2L  b_l = (1/d) (-r_T/d)^l sum_k C(k + l, k) (r_S/d)^k a_k       d = c_T - c_S
    L2L  b^C_l = sum_k C(k, l) rho^l tau^(k-l) b^P_k
with rho = r_C / r_P, tau = (c_C - c_P) / r_P.  The logarithmic potential of real
strengths is the real part of the integral: r sum_l b_l w^(l+1) / (l + 1) and a
constant per box, over a weak pair a_0 log|d| - Re sum_{k>=1} a_k (r_S/d)^k / k and
from the parent its series at the child's centre."""
import numpy as np


def _binom(n):
    c = np.zeros((n, n))
    c[:, 0] = 1.0
    for i in range(1, n):
        for k in range(1, i + 1):
            c[i, k] = c[i - 1, k - 1] + c[i - 1, k]
    return c


class Order:
    def __init__(self, orc, z, m, L, theta, p):
        self.z, self.m, self.L, self.p = z, m, L, p
        self.perm, self.range, geom = orc.tree(z, L)
        self.lists = orc.lists(geom, L, theta)
        self.c, self.r = geom[:, 4] + 1j * geom[:, 5], geom[:, 6]
        assert np.all(self.r > 0)
        self.base = [(4 ** l - 1) // 3 for l in range(L + 1)]
        C = _binom(2 * p)
        nb, lb = self.base[L], self.base[L - 1]
        self.a = np.zeros((nb, p), complex)
        self.b = np.zeros((nb, p), complex)
        self.const = np.zeros(nb)
        leaf = np.repeat(np.arange(lb, nb), self.range[lb:nb, 1])     # of the points in tree order
        zt, mt = z[self.perm], m[self.perm]
        t, w = mt.astype(complex), (zt - self.c[leaf]) / self.r[leaf]
        for k in range(p):
            np.add.at(self.a[:, k], leaf, t)
            t = t * w
        for l in range(L - 2, 0, -1):
            P = np.arange(self.base[l], self.base[l + 1])
            for q in range(4):
                ch = self.base[l + 1] + 4 * (P - self.base[l]) + q
                tau, rho = (self.c[ch] - self.c[P]) / self.r[P], self.r[ch] / self.r[P]
                tp = tau[:, None] ** np.arange(p)
                ac = self.a[ch] * rho[:, None] ** np.arange(p)
                for k in range(p):
                    self.a[P, k] += np.sum(C[k, :k + 1] * tp[:, k::-1][:, :k + 1] * ac[:, :k + 1], axis=1)
        K, M = np.arange(p), C[np.add.outer(np.arange(p), np.arange(p)), np.arange(p)[None, :]]
        for l in range(1, L):
            _, _, off, ids = self.lists[l]
            T = self.base[l] + np.repeat(np.arange(4 ** l), np.diff(off))
            S = self.base[l] + ids
            d = self.c[T] - self.c[S]
            X = self.a[S] * (self.r[S] / d)[:, None] ** K
            Y = (X @ M.T) * (-self.r[T] / d)[:, None] ** K / d[:, None]
            np.add.at(self.b, T, Y)
            lg = self.a[S, 0].real * np.log(np.abs(d))
            if p > 1:
                lg = lg - np.sum(X[:, 1:] / K[1:], axis=1).real
            np.add.at(self.const, T, lg)
        for l in range(1, L - 1):
            P = np.arange(self.base[l], self.base[l + 1])
            for q in range(4):
                ch = self.base[l + 1] + 4 * (P - self.base[l]) + q
                tau, rho = (self.c[ch] - self.c[P]) / self.r[P], self.r[ch] / self.r[P]
                tp = tau[:, None] ** np.arange(p + 1)
                self.const[ch] += self.const[P] + self.r[P] * np.sum(self.b[P] * tp[:, 1:] / (K + 1), axis=1).real
                for j in range(p):
                    self.b[ch, j] += rho ** j * np.sum(C[j:p, j] * tp[:, :p - j] * self.b[P, j:], axis=1)

    def _sources(self, g):
        """indices of the sources in the strong list of leaf g (local index)"""
        off, ids = self.lists[self.L - 1][:2]
        lb = self.base[self.L - 1]
        return np.concatenate([self.perm[s:s + n] for s, n in self.range[lb + ids[off[g]:off[g + 1]]]])

    def log(self):
        u, lb, K = np.zeros(self.z.size), self.base[self.L - 1], np.arange(self.p)
        for g in range(4 ** (self.L - 1)):
            s, n = self.range[lb + g]
            i, j = self.perm[s:s + n], self._sources(g)
            d = np.abs(self.z[i][:, None] - self.z[j])
            lg = np.log(np.where(d > 0, d, 1.0))
            w = (self.z[i] - self.c[lb + g]) / self.r[lb + g]
            far = self.r[lb + g] * np.sum(self.b[lb + g] * w[:, None] ** (K + 1) / (K + 1), axis=1).real
            u[i] = lg @ self.m[j].real + far + self.const[lb + g]
        return u

    def leaf_of(self, y):
        """the leaf (global box) that every point reaches, going down into the child whose
        disc holds it with the smallest |y - c| / r; -1 where it stops above"""
        box = np.zeros(y.size, np.int64)
        for l in range(self.L - 1):
            ch = self.base[l + 1] + 4 * (box - self.base[l])[:, None] + np.arange(4)
            q = np.abs(y[:, None] - self.c[ch]) / self.r[ch]
            k = np.argmin(q, axis=1)
            ok = (q[np.arange(y.size), k] <= 1.0) & (box >= self.base[l])
            box = np.where(ok, ch[np.arange(y.size), k], -1)
        return box

    def points(self, y, box):
        """field and derivative at y, every one in leaf box"""
        phi, dphi = np.zeros(y.size, complex), np.zeros(y.size, complex)
        K = np.arange(self.p)
        for g in np.unique(box):
            i, j = np.nonzero(box == g)[0], self._sources(g - self.base[self.L - 1])
            inv = 1.0 / (y[i][:, None] - self.z[j])
            w = ((y[i] - self.c[g]) / self.r[g])[:, None]
            phi[i] = inv @ self.m[j] + np.sum(self.b[g] * w ** K, axis=1)
            dphi[i] = -(inv * inv) @ self.m[j] + np.sum(self.b[g][1:] * K[1:] * w ** K[:-1], axis=1) / self.r[g]
        return phi, dphi

    def near(self, y, box):
        """the part of the field summed directly, and the distance to the nearest source"""
        out, dist = np.zeros(y.size, complex), np.zeros(y.size)
        for g in np.unique(box):
            i, j = np.nonzero(box == g)[0], self._sources(g - self.base[self.L - 1])
            d = y[i][:, None] - self.z[j]
            out[i], dist[i] = (1.0 / d) @ self.m[j], np.min(np.abs(d), axis=1)
        return out, dist
