"""Launch shapes chosen by the sizes of a call: results do not depend on them.

The per-receiver sums are formed in fixed chunks, so a receiver's numbers are
bitwise the same whichever receivers are solved with it and however the work
is dealt to the wavefronts.
"""
import numpy as np
import pytest

from paper_2507_04021_amd import scenes

pytestmark = pytest.mark.gpu

LOS, SPEC, DIFF = 1, 2, 4


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    import paper_2507_04021_amd as P
    P.lib()  # raises if the library is not built: no fallback
    return P


@pytest.fixture(scope="module")
def office(P):
    sc = scenes.office(seed=2507, target_points=60_000)
    return P.Scene.from_scene(sc, leaf_size=2, width=4)


def _solve(P, scene, rx, rays, K, **kw):
    r = P.solve(scene, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, 3.5e9, rays, K=K, flags=LOS | SPEC, **kw)
    return np.concatenate([t.cpu().numpy().reshape(len(rx), -1) for t in (r.gain, r.h_te, r.h_tm, r.parts)], 1), r


@pytest.mark.parametrize("pol", [None, ((1.0, 0.2, -0.3), (0.1, -1.0, 0.4))])
def test_refinement_slices_do_not_change_a_receiver(P, office, pol):
    """64 receivers have a refinement unit of 8 receivers for every wavefront; 9 and 1 do not, and get thinner units."""
    rx = scenes.office_rx()
    print("[gpu-test] refinement slices", flush=True)
    full, r = _solve(P, office, rx, 1 << 19, 4, pol=pol)
    assert r.counter("keys") > 4096 * 8 and r.counter("specular") > 0
    for take in (slice(0, 9), slice(5, 6), slice(61, 64)):
        part, _ = _solve(P, office, rx[take], 1 << 19, 4, pol=pol)
        assert np.array_equal(part, full[take])


@pytest.mark.parametrize("n", [1, 3, 257, 4096, 5000, 20_000, 66_000])
def test_ray_lanes_do_not_change_a_ray(P, office, n):
    """The first n rays of a budget, traced alone: small launches give a wavefront 4 to 32 rays, larger ones 64."""
    budget, K = 70_000, 3
    print("[gpu-test] ray lanes %d" % n, flush=True)
    _, full = _solve(P, office, scenes.office_rx()[:2], budget, K, want_seq=True)
    _, part = _solve(P, office, scenes.office_rx()[:2], budget, K, want_seq=True, ray_subset=np.arange(n))
    assert np.array_equal(part.seq.cpu().numpy(), full.seq.cpu().numpy()[:n])
    assert part.counter("rays") == n
    assert part.counter("interactions") == int((full.seq[:n] >= 0).sum())


@pytest.fixture(scope="module")
def room(P):
    sc = scenes.box_room(spacing=0.1, radius=0.08)
    return sc, P.Scene.from_scene(sc)


@pytest.mark.parametrize("rays,K", [(1, 1), (255, 2), (257, 3), (2000, 2), (9000, 3)])
def test_key_list_from_table_and_from_marks(P, room, rays, K):
    """A launch of every ray lists its keys from the table, the same rays as a subset from marked records."""
    print("[gpu-test] key list %d x %d" % (rays, K), flush=True)
    got = []
    for sub in (None, np.arange(rays)):
        r = P.solve(room[1], scenes.box_room_materials(), scenes.BOX_TX, [scenes.BOX_RX], 3.5e9, rays, K=K,
                    flags=LOS | SPEC | 8, ray_subset=sub)
        got.append(P.paths(r))
    assert got[0]["n_keys"] == got[1]["n_keys"] > 0
    for k in ("key_ray", "key_len", "key_seq", "valid", "length", "amp_te"):
        assert np.array_equal(got[0][k], got[1][k]), k


@pytest.mark.parametrize("rays,K", [(256, 1), (1024, 4), (1280, 4), (5200, 4)])
def test_record_sort_sizes(P, orc, room, rays, K):
    """Records of one LDS sort (up to 4 096) and of the device-wide one, against the oracle."""
    print("[gpu-test] record sort %d x %d" % (rays, K), flush=True)
    mats, rx = scenes.box_room_materials(scatter=0.3), [scenes.BOX_RX, (2.0, 1.0, 0.7)]
    r = P.solve(room[1], mats, scenes.BOX_TX, rx, 3.5e9, rays, K=K, flags=DIFF)
    ref = orc.solve(room[0], mats, scenes.BOX_TX, rx, 3.5e9, rays, K=K, flags=DIFF)
    assert np.max(np.abs(r.gain.cpu().numpy() / ref.G - 1)) < 1e-4


def test_batch_of_many_transmitters_matches_single_solves(P, room):
    """130 transmitters: items beyond the first launch of 96, key lists gathered over all of them."""
    print("[gpu-test] batch of 130", flush=True)
    tx, n = scenes.trajectory(seed=4021, n=130, min_rays=1, max_rays=3000)
    mats, rx = scenes.box_room_materials(scatter=0.2), [scenes.BOX_RX, (2.0, 1.0, 0.7)]
    b = P.solve_batch(room[1], mats, tx, n, rx, 3.5e9, K=2, flags=LOS | SPEC | DIFF)
    for i in range(0, 130, 7):
        r = P.solve(room[1], mats, tx[i], rx, 3.5e9, int(n[i]), K=2, flags=LOS | SPEC | DIFF)
        for x, y in ((b.gain, r.gain), (b.h_te, r.h_te), (b.parts, r.parts)):
            assert np.array_equal(x[i].cpu().numpy(), y.cpu().numpy()), i


@pytest.mark.parametrize("n", [2, 3, 4, 5, 33, 64, 65, 97])
def test_cfr_sample_counts_agree(P, n):
    """Sample k of n over a bandwidth is sample 2 k of 2 n - 1: responses and gradients of the two must agree (tiles
    of 4 samples, runs of 64; FP64 rounding of the phases, 500 cycles at most: 1e-11)."""
    import torch
    from paper_2507_04021_amd import diff
    print("[gpu-test] cfr n=%d" % n, flush=True)
    g = P.Scene.from_scene(scenes.box_room(spacing=0.1, radius=0.08, labels="surface"))
    mats = scenes.hidden_materials(7, 8, scatter=(0.1, 0.5))
    rx = np.array([scenes.BOX_RX, [2.0, 3.0, 2.0], [4.5, 0.7, 0.9]], np.float32)
    rec = diff.record(g, mats, scenes.BOX_TX, rx, 8e9, 700, K=2)
    gen = torch.Generator().manual_seed(n)
    w = torch.randn(3, n, 2, dtype=torch.complex128, generator=gen).cuda()
    out = []
    for fine in (False, True):
        m = torch.tensor(mats, dtype=torch.float64, device="cuda", requires_grad=True)
        h = diff.cfr(m, rec, 1.5e9, 2 * n - 1 if fine else n)
        h = h[:, ::2] if fine else h
        torch.sum(torch.real(h * w)).backward()
        out.append((h.detach(), m.grad))
    for a, b in zip(*out):
        assert float(torch.max(torch.abs(a - b)) / torch.max(torch.abs(a))) < 1e-7 if a.dtype == torch.float64 else \
            float(torch.max(torch.abs(a - b)) / torch.max(torch.abs(a))) < 1e-11
