"""Galerkin P1 near field by triangle pairs against the same near field entry by entry (the path
under a memory cap): odd numbers of frequencies, a second pass of outer points (n_galerkin = 6: 36
of them), few and many touching points."""
import numpy as np
import pytest

from gpu_common import context, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,L,ng,nt", [("hyp", 1, 5, 3), ("hyp", 5, 6, 4), ("adlp", 3, 6, 3), ("adlp", 6, 2, 5)])
def test_pairs_match_entries(kernel, L, ng, nt):
    """Sums of up to 6 nt^4 + ... FP64 products in another order: equal to 1e-12 of the largest entry."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, lshape_mesh
    xyz, tri = lshape_mesh(2)
    s = circle_frequencies(L, 10.0, 0.9)
    kw = dict(scheme="galerkin_p1", leaf_size=16, eps3d=1e-4, eps_aca=1e-6, n_galerkin=ng, n_touch=nt)
    ctx = gaca.Context(0)   # its own: a cap holds for the whole context
    capped = gaca.Problem(ctx, xyz, tri, s, max_device_bytes=32 << 30, **kw)
    by_entry = capped.build(kernel)
    by_pairs = gaca.Problem(context(), xyz, tri, s, **kw).build(kernel)
    _, near = capped.blocks()
    worst = top = 0.0
    for b, (_, m, _, n) in enumerate(near):
        e, p = by_entry.near_block(b, int(m), int(n)), by_pairs.near_block(b, int(m), int(n))
        worst, top = max(worst, np.abs(e - p).max()), max(top, np.abs(e).max())
    log(f"{kernel} L {L}: {len(near)} near blocks, largest difference {worst / top:.1e} of the largest entry")
    assert top > 0 and worst <= 1e-12 * top
