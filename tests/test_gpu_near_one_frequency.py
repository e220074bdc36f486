"""Near field where every frequency is the same: the disc of the frequencies has radius 0, at the origin
(the Laplace kernel at every frequency), next to it and away from it."""
import numpy as np
import pytest

from gpu_common import context, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme,kernel", [("collocation", "slp"), ("collocation", "dlp"), ("galerkin", "slp"),
                                           ("p1", "dlp")])
@pytest.mark.parametrize("s0", [0.0, 1e-300, 3.0])
def test_one_frequency(scheme, kernel, s0):
    """Every near block against the entries evaluated point by point, 1e-14 of the near field's
    largest (both are sums of at most 64 x 64 points, their order differs)."""
    import paper_2312_11219_amd as gaca
    from inputs import cube_mesh
    xyz, tri = cube_mesh(3)
    L = 16
    prob = gaca.Problem(context(), xyz, tri, np.full(L, s0, dtype=complex), scheme=scheme, leaf_size=16,
                        eps3d=1e-4, eps_aca=1e-6)
    h, (_, near), perm = prob.build(kernel), prob.blocks(), prob.perm
    worst, top = 0.0, 0.0
    for b in range(0, len(near), 3):
        r0, m, c0, n = (int(v) for v in near[b])
        got = np.transpose(h.near_block(b, m, n), (0, 2, 1))   # m x n x L
        i, j = (v.ravel() for v in np.meshgrid(np.arange(m), np.arange(n), indexing="ij"))
        ref = prob.eval_entries(kernel, perm[r0 + i], perm[c0 + j], np.zeros(i.size, int), np.zeros(i.size)).reshape(m, n, 1)
        assert np.isfinite(got).all()
        worst, top = max(worst, np.abs(got - ref).max()), max(top, np.abs(ref).max())
    log(f"{scheme} {kernel} s = {s0}: largest difference {worst:.1e} of {top:.1e}")
    assert worst <= 1e-14 * top
