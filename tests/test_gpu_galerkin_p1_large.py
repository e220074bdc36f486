"""Galerkin P1 near field by triangle pairs on meshes whose pairs exceed the buffer of their integrals: in
chunks of rows, against the near field entry by entry, and without a drop in speed as the mesh grows."""
import numpy as np
import pytest

from gpu_common import context, log

pytestmark = pytest.mark.gpu
KW = dict(scheme="galerkin_p1", leaf_size=16, eps3d=1e-3, eps_aca=1e-5, n_touch=3, n_galerkin=3)


@pytest.mark.parametrize("kernel", ["hyp", "adlp"])
def test_chunks_match_entries(kernel):
    """3072-triangle cube, 4.3 million pairs of triangles, three chunks: 1e-12 of the largest entry (sums
    in another order)."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh
    xyz, tri = cube_mesh(16)
    s = circle_frequencies(3, 10.0, 0.9)
    capped = gaca.Problem(gaca.Context(0), xyz, tri, s, max_device_bytes=64 << 30, **KW)   # its own context
    by_entry, by_pairs = capped.build(kernel), gaca.Problem(context(), xyz, tri, s, **KW).build(kernel)
    _, near = capped.blocks()
    worst = top = 0.0
    for b in range(0, len(near), 7):
        m, n = int(near[b][1]), int(near[b][3])
        e, p = by_entry.near_block(b, m, n), by_pairs.near_block(b, m, n)
        worst, top = max(worst, np.abs(e - p).max()), max(top, np.abs(e).max())
    log(f"{kernel}: {len(near)} near blocks, largest difference {worst / top:.1e} of the largest entry")
    assert top > 0 and worst <= 1e-12 * top


def test_time_grows_with_the_pairs():
    """From 3072 to 12288 triangles (4.3 to 19 million pairs) the near field takes at most four times as long
    per near entry (entry by entry it is over twenty times)."""
    import paper_2312_11219_amd as gaca
    from inputs import circle_frequencies, cube_mesh
    per = []
    for n in (16, 32):
        xyz, tri = cube_mesh(n)
        prob = gaca.Problem(context(), xyz, tri, circle_frequencies(2, 10.0, 0.9), **KW)
        entries = sum(int(b[1]) * int(b[3]) for b in prob.blocks()[1])
        ms = min(h.stats()["ms_near"] for h in [prob.build("hyp") for _ in range(2)])
        log(f"{len(tri)} triangles: {entries} near entries a frequency, {ms:.1f} ms")
        per.append(ms / entries)
    assert per[1] <= 4.0 * per[0]
