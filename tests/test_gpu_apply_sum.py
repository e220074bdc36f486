"""The reordered product (SUM) against the sum over the frequencies of the product at every frequency
(PER_FREQ, other kernels) of the same operator: more than 16 crosses per block, more than 128
columns (block columns, right-hand sides) in a far block, numbers of right-hand sides that are no
multiple of 4, leaves of more than 16 and 32 rows, a contraction that is no multiple of 16."""
import numpy as np
import pytest

from gpu_common import context, log, rel_fro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf,L,nrhs,eps,precision,dtype", [
    (12, 32, 34, 1, 1e-9, "fp64", "complex128"), (12, 16, 5, 3, 1e-4, "mixed", "complex128"),
    (6, 12, 16, 130, 1e-4, "fp64", "complex128"), (8, 48, 3, 2, 1e-5, "mixed", "complex64"),
    (5, 16, 64, 15, 1e-6, "fp64", "complex64"), (2, 16, 7, 1, 1e-4, "fp64", "complex128")])
def test_sum(n, leaf, L, nrhs, eps, precision, dtype):
    """Bars: 1e-12 in complex128, 2e-5 in complex64 (sums of some thousand FP32 products)."""
    import torch
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh, random_rhs
    xyz, tri = cube_mesh(n)
    prob = gaca.Problem(context(), xyz, tri, circle_frequencies(L, 25.0, 0.9), leaf_size=leaf, eps3d=eps,
                        eps_aca=0.1 * eps, precision=precision)
    h = prob.build("slp")
    X = torch.from_numpy(random_rhs(L, tri.shape[0], nrhs, seed=5)).cuda().to(getattr(torch, dtype))
    ref = h.apply(X, mode="per_freq").cpu().numpy().sum(0)
    got = h.apply(X).cpu().numpy()
    again = h.apply(X).cpu().numpy()
    st = h.stats()
    err = rel_fro(got, ref)
    far = prob.blocks()[0]
    log(f"n {n} leaf {leaf} L {L} nrhs {nrhs}: {far.shape[0]} far blocks, rank up to {st['rank_max']}: {err:.1e}")
    assert err < (1e-12 if dtype == "complex128" else 2e-5)
    assert np.array_equal(got, again)
