"""Recompression of faces with sides above 32 by rank: up to 32, up to 48 (in LDS, factors passing
through it 32 or 48 columns at a time) and above, against the oracle's QR and SVD."""
import numpy as np
import pytest

from gpu_common import context, log, reconstruct, rel_fro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,r", [(33, 64, 32), (200, 33, 30), (33, 33, 33), (96, 49, 48), (150, 300, 40),
                                   (49, 60, 49), (64, 130, 60), (40, 40, 2)])
def test_matches_oracle(m, n, r):
    """Faces with singular values 1 ... 1e-5 (the ACA keeps most of them): crosses, pivots and truncated face ranks are the
    oracle's, the tensor within 10 eps (the bar of the compression)."""
    import torch
    import paper_2312_11219_amd as gaca
    from oracle.aca3d import aca3d
    rng = np.random.default_rng(100 * m + n)
    L = 6

    def ortho(k):
        return np.linalg.qr(rng.standard_normal((k, r)) + 1j * rng.standard_normal((k, r)))[0]

    T = np.zeros((m, n, L), dtype=complex)
    for p in range(2):
        H = (ortho(m) * np.logspace(0, -5, r)[None, :]) @ ortho(n).T
        T += 0.1 ** p * H[:, :, None] * (rng.standard_normal(L) + 1j * rng.standard_normal(L))[None, None, :]
    eps, eps_aca = 1e-4, 1e-6
    h = gaca.compress_tensor(context(), torch.from_numpy(T).cuda(), eps3d=eps, eps_aca=eps_aca, recompress=1)
    b, o = h.export_block(0), aca3d(T, eps, eps_aca, recompress_faces=True)
    err = rel_fro(reconstruct(h, 0), T)
    log(f"{m} x {n}: face ranks {[c['rho'] for c in b['crosses']]} (oracle {[c.U.shape[1] for c in o.crosses]}), error {err:.1e}")
    assert err < 10 * eps and b["rank"] == o.rank
    assert [(c["k"], c["i"], c["j"], c["rho"]) for c in b["crosses"]] == \
        [(c.k, c.i, c.j, c.U.shape[1]) for c in o.crosses]
