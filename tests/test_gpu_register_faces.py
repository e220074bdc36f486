"""Faces held in registers through their ACA: every size class of the kernel at its edges (one
row or column short of, at and past the largest side; one long side), zero rows on the way,
against the oracle; the FP32 classes on far blocks of all sides up to 192."""
import numpy as np
import pytest

from gpu_common import context, log, reconstruct, rel_fro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(24, 23), (25, 24), (32, 31), (33, 40), (41, 48), (7, 48), (49, 64), (65, 12),
                                 (80, 79), (81, 96), (3, 97), (128, 127), (129, 150), (160, 159), (161, 40)])
def test_classes_match_oracle(m, n):
    """Known-rank tensors with rows of zeros: exact reconstruction (rounding of sums of rank 6 in
    FP64, bar 1e-11) and the oracle's pivots."""
    import torch
    import paper_2312_11219_amd as gaca
    from oracle.aca3d import aca3d
    rng = np.random.default_rng(1000 * m + n)
    L, R, rho = 5, 2, min(6, m, n) // 2 + 1
    T = np.zeros((m, n, L), dtype=complex)
    for _ in range(R):
        H = (rng.standard_normal((m, rho)) + 1j * rng.standard_normal((m, rho))) @ \
            (rng.standard_normal((rho, n)) + 1j * rng.standard_normal((rho, n)))
        H[[0, m // 2]] = 0.0
        T += H[:, :, None] * (rng.standard_normal(L) + 1j * rng.standard_normal(L))[None, None, :]
    h = gaca.compress_tensor(context(), torch.from_numpy(T).cuda(), eps3d=1e-10, eps_aca=1e-12)
    b, o = h.export_block(0), aca3d(T, 1e-10, 1e-12)
    err = rel_fro(reconstruct(h, 0), T)
    log(f"face {m} x {n}: rank {b['rank']}, face ranks {[c['rho'] for c in b['crosses']]}, error {err:.1e}")
    assert b["rank"] == o.rank and err < 1e-11
    assert [(c["k"], c["i"], c["j"]) for c in b["crosses"]] == [(c.k, c.i, c.j) for c in o.crosses]
    assert [c["rho"] for c in b["crosses"]] == [c.U.shape[1] for c in o.crosses]


def test_mixed_sides_up_to_192():
    """3072-triangle cube with leaves of 192 and of 24 elements: FP32 faces of 192, 96, 48 and 24
    rows.  Each sampled block's error exceeds the FP64 build's by at most 1e-5 (the mixed path's
    bar)."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh
    from oracle.hmatrix import Problem
    xyz, tri = cube_mesh(16)
    s = circle_frequencies(8, 20.0, 0.95)
    for leaf in (192, 24):
        op = Problem(xyz, tri, s, leaf, 1.0)
        hs = [gaca.Problem(context(), xyz, tri, s, leaf_size=leaf, eps3d=1e-5, eps_aca=1e-7,
                           precision=p).build("slp") for p in ("fp64", "mixed")]
        sides = [max(b[1], b[3]) for b in op.far]
        pick = [b for side in sorted(set(sides)) for b in [i for i, v in enumerate(sides) if v == side][:4]]
        for b in pick:
            T = op.block_tensor("slp", op.far[b], True)
            e64, emx = (rel_fro(reconstruct(h, b), T) for h in hs)
            log(f"leaf {leaf} block {b} ({op.far[b][1]} x {op.far[b][3]}): fp64 {e64:.1e} mixed {emx:.1e}")
            assert emx - e64 <= 1e-5
