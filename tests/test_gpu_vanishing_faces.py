"""Double layer on meshes of flat pieces: faces with entries that vanish between coplanar elements
leave the register kernels above sides of 64 (from there the kernel in HBM takes them), faces
without go on in registers."""
import numpy as np
import pytest

from gpu_common import context, log, rel_fro, reconstruct

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["dlp", "both"])
def test_flat_pieces(kernel):
    """Far blocks with a side of 65 to 160, every fifth: error against the far entries within the tolerance
    (eps3d with the usual factor 10 between a block's stop estimate and its error)."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh
    xyz, tri = cube_mesh(21)   # 5292 triangles: clusters of 82 and 83 beside larger and smaller ones
    L, eps = 12, 1e-5
    prob = gaca.Problem(context(), xyz, tri, circle_frequencies(L, 10.0, 0.9), leaf_size=16, eps3d=eps, eps_aca=1e-6)
    h = prob.build_both()[1] if kernel == "both" else prob.build("dlp")
    far, perm = prob.blocks()[0], prob.perm
    worst, kinds = 0.0, [0, 0]
    pick = [b for b, blk in enumerate(far) if 64 < max(blk[1], blk[3]) <= 160][::5]
    for b in pick:
        r0, m, c0, n = far[b]
        i, j, k = (v.ravel() for v in np.meshgrid(np.arange(m), np.arange(n), np.arange(L), indexing="ij"))
        T = prob.eval_entries("dlp", perm[r0 + i], perm[c0 + j], k, np.ones(i.size)).reshape(m, n, L)
        if not T.any():
            continue
        kinds[int((np.abs(T[:, :, 0]) < 1e-13 * np.abs(T[:, :, 0]).max()).any())] += 1
        worst = max(worst, rel_fro(reconstruct(h, b), T))
    log(f"{kernel}: {kinds[0]} blocks without and {kinds[1]} with vanishing entries, worst error {worst:.1e}")
    assert kinds[1] > 0 and worst < 10 * eps


@pytest.mark.parametrize("m,n", [(65, 80), (96, 90), (128, 97), (160, 159)])
def test_full_faces_match_oracle(m, n):
    """Known-rank tensors without vanishing entries: the oracle's pivots and ranks, error 1e-11."""
    import torch
    import paper_2312_11219_amd as gaca
    from oracle.aca3d import aca3d
    rng = np.random.default_rng(m + n)
    T = np.zeros((m, n, 4), dtype=complex)
    for _ in range(2):
        H = (rng.standard_normal((m, 3)) + 1j * rng.standard_normal((m, 3))) @ \
            (rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n)))
        T += H[:, :, None] * (rng.standard_normal(4) + 1j * rng.standard_normal(4))[None, None, :]
    h = gaca.compress_tensor(context(), torch.from_numpy(T).cuda(), eps3d=1e-10, eps_aca=1e-12)
    b, o = h.export_block(0), aca3d(T, 1e-10, 1e-12)
    assert rel_fro(reconstruct(h, 0), T) < 1e-11
    assert [(c["k"], c["i"], c["j"], c["rho"]) for c in b["crosses"]] == \
        [(c.k, c.i, c.j, c.U.shape[1]) for c in o.crosses]
