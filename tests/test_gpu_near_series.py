"""Near field from the power series in the frequency against the entries evaluated point by point at
every frequency: every scheme and class of pairs, 24, 32 and 44 terms, pairs on both sides of the
series' bound (many wavelengths per element), fewer frequencies than lanes, no conjugate symmetry."""
import numpy as np
import pytest

from gpu_common import context, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme,kernel,precision,L,c0,sym", [
    ("galerkin", "slp", "fp64", 16, 4.0, True), ("galerkin", "slp", "fp64", 17, 7.0, True),
    ("galerkin", "slp", "mixed", 33, 12.0, True), ("galerkin", "slp", "fp64", 9, 30.0, False),
    ("collocation", "slp", "fp64", 24, 8.0, True), ("collocation", "dlp", "fp64", 16, 16.0, True),
    ("collocation", "dlp", "mixed", 9, 40.0, False), ("p1", "dlp", "fp64", 16, 6.0, True),
    ("p1", "dlp", "fp64", 31, 14.0, False)])
def test_series_matches_points(scheme, kernel, precision, L, c0, sym):
    """Of the block's largest entry at the frequency: 1e-12 (FP64; the terms of the series exceed
    its sum by up to e^6 = 400), 1e-6 (stored in FP32)."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, lshape_mesh
    xyz, tri = lshape_mesh(3)
    xyz = xyz + 0.02 * np.sin(17.0 * xyz + np.arange(3))   # no two triangles alike
    s = circle_frequencies(L, c0, 0.9)
    if not sym:
        s = s * np.exp(0.05j)
    prob = gaca.Problem(context(), xyz, tri, s, scheme=scheme, leaf_size=16, eps3d=1e-4, eps_aca=1e-6,
                        precision=precision)
    h = prob.build(kernel)
    _, near = prob.blocks()
    rng = np.random.default_rng(1)
    perm = prob.perm
    worst = 0.0
    for b in rng.permutation(len(near))[:40]:
        r0, m, c0_, n = (int(v) for v in near[b])
        got = np.transpose(h.near_block(int(b), m, n), (0, 2, 1))   # m x n x L
        i, j, k = (v.ravel() for v in np.meshgrid(np.arange(m), np.arange(n), np.arange(L), indexing="ij"))
        ref = prob.eval_entries(kernel, perm[r0 + i], perm[c0_ + j], k, np.zeros(i.size)).reshape(m, n, L)
        top = np.abs(ref).max((0, 1))
        assert np.isfinite(got).all()
        worst = max(worst, (np.abs(got - ref).max((0, 1)) / np.maximum(top, 1e-300)).max())
    log(f"{scheme} {kernel} {precision} L {L} c0 {c0}: largest difference {worst:.1e}")
    assert worst <= (1e-12 if precision == "fp64" else 1e-6)
