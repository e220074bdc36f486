"""The product at every frequency (PER_FREQ, matrix cores) summed over the frequencies against the
reordered product (SUM, other kernels) of the same operator: column counts that are no multiple of
16 or 64, leaves of more than 32 rows, every storage and right-hand-side type, a mesh without far
blocks."""
import numpy as np
import pytest

from gpu_common import context, log, rel_fro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf,L,nrhs,precision,dtype", [
    (4, 8, 5, 1, "fp64", "complex128"), (4, 40, 9, 2, "fp64", "complex128"), (8, 16, 16, 4, "fp64", "complex128"),
    (6, 8, 33, 5, "mixed", "complex128"), (6, 48, 3, 7, "mixed", "complex64"), (5, 16, 64, 1, "fp64", "complex64"),
    (2, 16, 7, 3, "fp64", "complex128")])
def test_sum_over_frequencies(n, leaf, L, nrhs, precision, dtype):
    """Bars: 1e-12 in complex128, 2e-5 in complex64 (sums of some thousand FP32 products)."""
    import torch
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh, random_rhs
    xyz, tri = cube_mesh(n)
    prob = gaca.Problem(context(), xyz, tri, circle_frequencies(L, 10.0, 0.9), leaf_size=leaf, eps3d=1e-4,
                        eps_aca=1e-6, precision=precision)
    h = prob.build("dlp")
    X = torch.from_numpy(random_rhs(L, tri.shape[0], nrhs, seed=3)).cuda().to(getattr(torch, dtype))
    ref = h.apply(X).cpu().numpy()
    got = h.apply(X, mode="per_freq").cpu().numpy()
    one = torch.zeros_like(X)
    one[L // 2] = X[L // 2]
    err = rel_fro(got.sum(0), ref)
    err1 = rel_fro(got[L // 2], h.apply(one).cpu().numpy())
    log(f"n {n} leaf {leaf} L {L} nrhs {nrhs}: {prob.blocks()[0].shape[0]} far blocks, {err:.1e}, one frequency {err1:.1e}")
    assert max(err, err1) < (1e-12 if dtype == "complex128" else 2e-5)
