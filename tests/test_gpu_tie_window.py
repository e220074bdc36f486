"""A wide tie window: the pivot may be a small entry of its row, so that w has entries up to 1 / (1 - tie),
and the stopping test has to know it."""
import numpy as np
import pytest

from gpu_common import context, log, rel_fro, reconstruct

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tie", [0.5, 0.9])
@pytest.mark.parametrize("m,n", [(20, 22), (40, 33), (60, 64), (79, 80), (96, 90), (128, 120)])
def test_ranks_match_oracle(m, n, tie):
    """Rank-one terms of flat magnitude 1, d, d^2, the first row's first entry just within the window of the
    first, and a tolerance that the second step just meets: |u||w| = 0.95 eps |S|, but above eps times the |S|
    that |w_j| <= 1 would bound.  The oracle's pivots and face ranks."""
    import torch
    import paper_2312_11219_amd as gaca
    from oracle.aca3d import aca3d, face_aca
    rng = np.random.default_rng(m + n)
    H = np.zeros((m, n), dtype=complex)
    for k in range(3):
        a, b = (np.exp(2j * np.pi * rng.random(v)) for v in (m, n))
        if k == 0:
            b[0] *= 1.3 * (1.0 - tie)
        H += 1e-3 ** k * a[:, None] * b[None, :]
    U, W = face_aca(H, 0.0, 0.0, 2, tie)[:2]
    S = np.linalg.norm(U @ W.T)
    eps_aca = np.linalg.norm(U[:, 1]) * np.linalg.norm(W[:, 1]) / (0.95 * S)
    assert np.sqrt(m * n) * np.abs(U).max(0).sum() < 0.9 * S
    T = H[:, :, None] * np.array([1.0, 0.5j])[None, None, :]
    h = gaca.compress_tensor(context(), torch.from_numpy(T).cuda(), eps3d=0.1, eps_aca=eps_aca, tie=tie)
    b, o = h.export_block(0), aca3d(T, 0.1, eps_aca, tie=tie)
    got, ref = ([(c["k"], c["i"], c["j"], c["rho"]) for c in b["crosses"]],
                [(c.k, c.i, c.j, c.U.shape[1]) for c in o.crosses])
    log(f"{m} x {n} tie {tie}: {got} oracle {ref} error {rel_fro(reconstruct(h, 0), T):.1e}")
    assert got == ref
