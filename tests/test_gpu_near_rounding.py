"""Near field of coarse meshes (a few wavelengths and decay lengths per element) against the same
quadrature in 80-bit arithmetic: no digits beyond the rounding of the points' own sum are lost."""
import numpy as np
import pytest

from gpu_common import context, log

pytestmark = pytest.mark.gpu
LD = np.longdouble


def _rules():
    from oracle.quadrature import gauss01, triangle6

    def collapsed(n):
        x, w = gauss01(n)
        u, v = (z.ravel() for z in np.meshgrid(x, x, indexing="ij"))
        return np.stack([1 - u, u * (1 - v), u * v], 1), 2.0 * np.outer(w * x, w).ravel()

    return [triangle6(), collapsed(4), collapsed(8)]


@pytest.mark.parametrize("Rrad", [0.5, 2.0, 5.5])
@pytest.mark.parametrize("scheme,kernel", [("collocation", "slp"), ("collocation", "dlp"), ("galerkin", "slp")])
def test_rounding(scheme, kernel, Rrad):
    """One near block of all elements, disjoint pairs of every class but the close Galerkin ones: error of each
    entry within (2 |s| r + 40) 2^-53 of the sum of its terms' magnitudes (r and s r rounded, a handful
    of products per term, 64 terms of one sign added).  Rrad: radius of the frequencies times the radius of the
    largest triangle (Galerkin: two triangles)."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh
    xyz, tri = cube_mesh(3)
    xyz = xyz + 0.02 * np.sin(17.0 * xyz + np.arange(3))   # no two triangles alike
    V = xyz[tri]
    cen, M, L = V.mean(1), len(tri), 40
    h = np.stack([np.linalg.norm(V[:, a] - V[:, a - 1], axis=1) for a in range(3)]).max(0)
    rad = np.linalg.norm(V - cen[:, None], axis=2).max() * (2 if scheme == "galerkin" else 1)
    s = circle_frequencies(L, Rrad / rad / 0.9, 0.9)
    prob = gaca.Problem(context(), xyz, tri, s, scheme=scheme, leaf_size=M, eps3d=1e-4, eps_aca=1e-6)
    hm, (_, near), perm = prob.build(kernel), prob.blocks(), np.asarray(prob.perm)
    assert len(near) == 1 and near[0][1] == M
    got = np.empty((M, M, L), complex)
    got[np.ix_(perm, perm)] = np.transpose(hm.near_block(0, M, M), (0, 2, 1))
    nrm = np.cross(V[:, 1] - V[:, 0], V[:, 2] - V[:, 0])
    area = 0.5 * np.linalg.norm(nrm, axis=1)
    nrm = nrm / (2 * area[:, None])
    dist = np.linalg.norm(cen[:, None] - cen[None], axis=2)
    q = dist / (np.maximum(h[:, None], h[None]) if scheme == "galerkin" else h[None])
    touch = (tri[:, None, :, None] == tri[None, :, None, :]).any((2, 3))
    tier = np.where(q >= 4, 0, np.where(q >= 2, 1, 2))
    tier[(touch if scheme == "galerkin" else np.eye(M, dtype=bool)) | ((tier == 2) & (scheme == "galerkin"))] = -1
    rng = np.random.default_rng(3)
    worst = {}
    sL = s.astype(np.clongdouble)
    for t, (lam, w) in enumerate(_rules()):
        ij = np.argwhere(tier == t)
        for i, j in ij[rng.permutation(len(ij))[:60]]:
            Y, wy = lam @ V[j], w * area[j]
            if scheme == "galerkin":
                X = np.repeat(lam @ V[i], len(w), 0)
                Y, wt = np.tile(Y, (len(w), 1)), np.outer(w * area[i], wy).ravel()
            else:
                X, wt = cen[i][None], wy
            d = X.astype(LD) - Y.astype(LD)
            r = np.sqrt((d * d).sum(1))
            k = wt.astype(LD) / (4 * np.arccos(LD(-1)) * r)
            f = 1
            if kernel == "dlp":
                k, f = k * ((d * nrm[j].astype(LD)).sum(1) / r ** 2), 1 + sL[:, None] * r
                if np.abs(k).max() * r.max() < 1e-6 * area[j] / r.max():
                    continue   # x_i nearly in the triangle's plane: n (x - y) cancels
            term = k * f * np.exp(-sL[:, None] * r)
            err = np.abs(got[i, j] - term.sum(1)) / np.abs(term).sum(1)
            bar = (2 * np.abs(s) * float(r.max()) + 40) * 2.0 ** -53
            if kernel == "dlp":   # the distance from the plane is a difference of coordinates
                bar = bar + 4 * 2.0 ** -53 / (np.abs(((cen[i] - V[j, 0]) * nrm[j]).sum()) + 1e-300)
            worst[t] = max(worst.get(t, (0, 0)), ((err / bar).max(), float(err.max())))
    log(f"{scheme} {kernel} R rad {Rrad}: worst of the bar and error by class " +
        ", ".join(f"{t}: {a:.2f} {e:.1e}" for t, (a, e) in worst.items()))
    assert worst and max(a for a, _ in worst.values()) <= 1.0


@pytest.mark.parametrize("scheme,kernel", [("collocation", "slp"), ("collocation", "dlp"), ("galerkin", "slp"),
                                           ("p1", "dlp")])
@pytest.mark.parametrize("left", [0.0, -6.0])
def test_scattered_frequencies(scheme, kernel, left):
    """Frequencies in no order, some twice, real ones, with real parts from `left` to 14: bands of one frequency
    and of many.  Every near block against the entries point by point, 1e-13 of the block's largest at the
    frequency (the bar of each side, (2 |s| r + 40) 2^-53, is below 2e-14 of the sum of the magnitudes)."""
    import paper_2312_11219_amd as gaca
    from inputs import lshape_mesh
    rng = np.random.default_rng(8)
    xyz, tri = lshape_mesh(3)
    xyz = xyz + 0.02 * np.sin(17.0 * xyz + np.arange(3))
    s = rng.uniform(left, 14.0, 27) + 1j * rng.uniform(-9.0, 9.0, 27)
    s[5], s[11], s[12], s[20] = s[2], 14.0, left, s[3].real
    prob = gaca.Problem(context(), xyz, tri, s, scheme=scheme, leaf_size=16, eps3d=1e-4, eps_aca=1e-6)
    h, (_, near), perm = prob.build(kernel), prob.blocks(), prob.perm
    worst = 0.0
    for b in rng.permutation(len(near))[:40]:
        r0, m, c0, n = (int(v) for v in near[b])
        got = np.transpose(h.near_block(int(b), m, n), (0, 2, 1))
        i, j, k = (v.ravel() for v in np.meshgrid(np.arange(m), np.arange(n), np.arange(len(s)), indexing="ij"))
        ref = prob.eval_entries(kernel, perm[r0 + i], perm[c0 + j], k, np.zeros(i.size)).reshape(m, n, len(s))
        worst = max(worst, (np.abs(got - ref).max((0, 1)) / np.maximum(np.abs(ref).max((0, 1)), 1e-300)).max())
    log(f"{scheme} {kernel} real parts from {left}: largest difference {worst:.1e}")
    assert worst <= 1e-13
