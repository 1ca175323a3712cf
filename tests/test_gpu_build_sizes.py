"""Hierarchy builds at the edges of the builder's launches: one block's tail (1 024 clusters), tiles of 1 012 clusters,
passes of 1 024 nodes, both builders and all widths. Every answer of a solve is independent of the hierarchy, so each scene's
results on the radix tree and on wider nodes must equal those on the clustering tree's binary nodes bitwise."""
import numpy as np
import pytest

from paper_2507_04021_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    import paper_2507_04021_amd as P
    P.lib()  # raises if the library is not built: no fallback
    return P


def _scene(n, grid):
    if grid:  # equal merged areas everywhere: ties decide, few pairs merge per pass
        k = int(round(n ** 0.5))
        return scenes.plane_patch(-1.0, 1.0, -1.0, 1.0, 2.0 / k, 1.5 / k)
    return scenes.random_disks(n, seed=n, extent=1.5, radius=min(0.25, 2.0 / n ** 0.5))


@pytest.mark.parametrize("n,grid", [(100, False), (257, False), (1024, False), (1025, False), (1300, False),
                                    (9000, False), (30_000, False), (1024, True), (4900, True)])
def test_build_sizes(P, n, grid):
    sc = _scene(n, grid)
    mats = np.tile([4.0, 0.05, 0.3], (3, 1))
    base = None
    for builder, width in ((2, 2), (2, 4), (2, 8), (1, 4)):
        print("[gpu-test] build n=%d grid=%d builder=%d width=%d" % (n, grid, builder, width), flush=True)
        g = P.Scene.from_scene(sc, leaf_size=2, width=width, builder=builder)
        assert g.info["stack_entries"] <= 96 and g.info["depth"] >= np.log2(n) - 1
        r = P.solve(g, mats, [0.05, -0.02, 0.61], [[0.3, 0.2, 0.5], [-0.4, 0.1, 0.9]], 3.5e9, 2000, K=2, flags=7,
                    want_seq=True)
        got = [x.cpu().numpy() for x in (r.seq, r.gain, r.h_te, r.parts)]
        base = base or got
        assert all(np.array_equal(a, b) for a, b in zip(got, base))


@pytest.mark.parametrize("rho", [0.05, 0.5, 8.0])
def test_point_sets_sort_the_bits_of_the_scene(P, rho):
    """Reception points against the mean of each voxel's points, voxels in index order (8 m: one voxel per octant)."""
    sc = scenes.random_disks(5000, seed=3, extent=1.5, radius=0.02)
    print("[gpu-test] point sets rho=%g" % rho, flush=True)
    g = P.Scene.from_scene(sc, dps_voxel=rho)
    vox = np.floor(sc.pos.astype(np.float64) / float(np.float32(rho))).astype(np.int64) + (1 << 20)
    _, of, cnt = np.unique(vox[:, 0] << 42 | vox[:, 1] << 21 | vox[:, 2], return_inverse=True, return_counts=True)
    want = np.stack([np.bincount(of, sc.pos[:, a].astype(np.float64)) / cnt for a in range(3)], 1)
    got = P.reception_points(g).cpu().numpy()
    assert got.shape == want.shape
    assert np.max(np.abs(got - want)) <= 2.0 ** -23 * 1.5  # one FP32 rounding of coordinates up to 1.5


@pytest.mark.parametrize("n", [1012, 1013, 2024, 2025, 3037, 70_001, 300_001])
def test_build_sizes_at_the_edges_of_a_tile(P, n):
    """A block of a clustering pass takes 1 012 clusters (the look-back goes past one tile from 1 013 on, past the 64 that
    one look covers from 64 769 on; a level of the wide collapse, in tiles of 256 nodes, in the largest); results as on the
    radix tree, bitwise."""
    sc = _scene(n, False)
    mats = np.tile([4.0, 0.05, 0.3], (3, 1))
    base = None
    for builder, width in ((1, 4), (2, 4), (2, 2), (2, 8)):
        print("[gpu-test] build n=%d builder=%d width=%d" % (n, builder, width), flush=True)
        g = P.Scene.from_scene(sc, leaf_size=2, width=width, builder=builder)
        r = P.solve(g, mats, [0.05, -0.02, 0.61], [[0.3, 0.2, 0.5], [-0.4, 0.1, 0.9]], 3.5e9, 2000, K=2, flags=7,
                    want_seq=True)
        got = [x.cpu().numpy() for x in (r.seq, r.gain, r.h_te, r.parts)]
        base = base or got
        assert all(np.array_equal(a, b) for a, b in zip(got, base))
