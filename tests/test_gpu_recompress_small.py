"""Recompression of small faces (one workgroup in LDS per face up to 32 x 32) at the edges of its two
sizes and just above them, against the oracle's QR and SVD."""
import numpy as np
import pytest

from gpu_common import context, log, reconstruct, rel_fro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(24, 24), (23, 5), (2, 24), (25, 24), (32, 32), (31, 9), (33, 32)])
def test_matches_oracle(m, n):
    """Faces with singular values 1 ... 1e-9: crosses, pivots and truncated face ranks are the
    oracle's, the tensor within 10 eps (the bar of the compression)."""
    import torch
    import paper_2312_11219_amd as gaca
    from oracle.aca3d import aca3d
    rng = np.random.default_rng(100 * m + n)
    L, r = 6, min(m, n)

    def ortho(k):
        return np.linalg.qr(rng.standard_normal((k, r)) + 1j * rng.standard_normal((k, r)))[0]

    T = np.zeros((m, n, L), dtype=complex)
    for p in range(2):
        H = (ortho(m) * np.logspace(0, -9, r)[None, :]) @ ortho(n).T
        T += 0.1 ** p * H[:, :, None] * (rng.standard_normal(L) + 1j * rng.standard_normal(L))[None, None, :]
    eps, eps_aca = 1e-4, 1e-6
    h = gaca.compress_tensor(context(), torch.from_numpy(T).cuda(), eps3d=eps, eps_aca=eps_aca, recompress=1)
    b, o = h.export_block(0), aca3d(T, eps, eps_aca, recompress_faces=True)
    err = rel_fro(reconstruct(h, 0), T)
    log(f"{m} x {n}: face ranks {[c['rho'] for c in b['crosses']]} (oracle {[c.U.shape[1] for c in o.crosses]}), error {err:.1e}")
    assert err < 10 * eps and b["rank"] == o.rank
    assert [(c["k"], c["i"], c["j"], c["rho"]) for c in b["crosses"]] == \
        [(c.k, c.i, c.j, c.U.shape[1]) for c in o.crosses]
