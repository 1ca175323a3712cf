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


@pytest.mark.parametrize("n,n_labels", [(1, 1), (127, 8), (128, 16), (129, 17), (2049, 64), (32769, 8)])
def test_mlp_gradients_at_the_edges_of_a_block(P, n, n_labels):
    """A block takes 128 rows at a time, at most 256 blocks do, and labels are taken 16 at a time. The bar is that of
    the kernel against the reference at its rounding points: (2^-8 + n 2^-24) of the sum of |terms|."""
    import torch
    from oracle import mlp as R
    from paper_2507_04021_amd import mlp as M
    rng = np.random.default_rng(n)
    params = R.init_params(n_labels, seed=3)
    labels = rng.integers(0, n_labels, n)
    cosv = rng.uniform(0.0, 1.0, n).astype(np.float32)
    g_out = rng.normal(size=(n, 8)).astype(np.float32)
    g_out[:, 5:] = 0
    net = M.MaterialMLP(params)
    lab, cs = torch.tensor(labels.astype(np.int16), device="cuda"), torch.tensor(cosv, device="cuda")
    grads = net.backward_rows(lab, cs, 28e9, torch.tensor(g_out, device="cuda"))
    ref, mag = R.backward(params, labels, cosv.astype(np.float64), 28e9, g_out[:, :5], precision="kernel",
                          magnitudes=True)
    for k, v in ref.items():
        got = grads[k].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - v) <= (2.0 ** -8 + n * 2.0 ** -24) * mag[k]), k


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_mlp_row_without_a_finite_gradient_reaches_its_own_label_only(P, bad):
    import torch
    from oracle import mlp as R
    from paper_2507_04021_amd import mlp as M
    params = R.init_params(20, seed=4)
    net = M.MaterialMLP(params)
    n = 200
    labels = np.arange(n) % 20
    g = np.ones((n, 8), np.float32)
    lab = torch.tensor(labels.astype(np.int16), device="cuda")
    cs = torch.linspace(0, 1, n, device="cuda")
    ref = net.backward_rows(lab, cs, 28e9, torch.tensor(g, device="cuda"))["emb"].cpu().numpy()
    g[37, 0] = bad
    got = net.backward_rows(lab, cs, 28e9, torch.tensor(g, device="cuda"))["emb"].cpu().numpy()
    assert not np.isfinite(got[17]).any()
    keep = np.arange(20) != 17
    # the same sums in another order: 10 rows of a label, each addition off by at most 2^-24 of the sum of |terms|
    g[37, 0] = 1
    _, mag = R.backward(params, labels, cs.cpu().numpy().astype(np.float64), 28e9, g[:, :5], precision="kernel",
                        magnitudes=True)
    assert np.all(np.abs(got - ref)[keep] <= 20 * 2.0 ** -24 * mag["emb"][keep])


def test_mlp_forward_rows_do_not_depend_on_the_batch(P):
    """Few rows take one tile per wavefront, many take eight: a row's outputs are bitwise the same."""
    import torch
    from oracle import mlp as R
    from paper_2507_04021_amd import mlp as M
    net = M.MaterialMLP(R.init_params(8, seed=5))
    n = 300_000
    lab = torch.tensor((np.arange(n) * 7 % 9).astype(np.int16), device="cuda")
    cs = torch.rand(n, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    big, small = torch.zeros(n, 8, device="cuda"), torch.zeros(1000, 8, device="cuda")
    net.forward_rows(lab, cs, 28e9, big)
    net.forward_rows(lab[:1000], cs[:1000], 28e9, small)
    assert torch.equal(big[:1000], small)


@pytest.mark.parametrize("n_rx,n_edges", [(1, 1), (3, 5), (1, 17), (13, 40)])
def test_diffraction_lanes_per_pair_agree(P, office, n_rx, n_edges):
    """Up to 24 576 pairs take four lanes each, more take one. A pair's FP64 steps are the same up to the contraction of
    products and sums, which its series may blow up to 1e-9 of the amplitude: at most one rounding of the FP32 result
    apart. The sums of a receiver add at most 2^-52 of the terms' magnitudes per edge."""
    edges = scenes.office_edges(scenes.office(seed=2507, target_points=60_000))
    edges = (edges[0][:n_edges], edges[1][:n_edges])
    rx = scenes.office_rx()[:n_rx]
    out, amp = P.diffraction(office, edges, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, 3.5e9, want_pairs=True)
    reps = 24_576 // (n_rx * n_edges) + 1
    big, bamp = P.diffraction(office, edges, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, np.tile(rx, (reps, 1)), 3.5e9,
                              want_pairs=True)
    bamp = np.asarray(bamp)[-n_rx:]
    assert np.array_equal(amp != 0, bamp != 0)
    for part in (np.real, np.imag):
        assert np.all(np.abs(part(amp) - part(bamp)) <= 2.0 ** -23 * np.abs(amp))
    tol = (2.0 ** -22 + n_edges * 2.0 ** -52) * np.abs(amp).sum((1, 2))
    d = np.abs(out.cpu().numpy() - big.cpu().numpy()[-n_rx:])
    assert np.all(d[:, 1:] <= tol[:, None]) and np.all(d[:, 0] <= tol * np.abs(amp).max())


@pytest.mark.parametrize("n_rx", [1, 63, 65, 130])
def test_point_set_sums_do_not_depend_on_the_other_receivers(P, n_rx):
    """The visibility matrix is read in words of 64 receivers: a receiver's sums are bitwise those of a call of its own."""
    import torch
    sc = scenes.office(seed=2507, target_points=60_000)
    g = P.Scene.from_scene(sc, leaf_size=2, width=4, dps_voxel=0.3)
    rng = np.random.default_rng(n_rx)
    base = scenes.office_rx()
    rx = (base[rng.integers(0, len(base), n_rx)] + rng.uniform(-0.2, 0.2, (n_rx, 3))).astype(np.float32)
    vis = P.visibility(g, rx)
    kw = dict(K=3, flags=LOS | SPEC | DIFF | P.DPS_LAUNCH)
    n = g.info["n_point_sets"]

    def rows(i):
        r = P.solve(g, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx[i], 3.5e9, n, dps_vis=vis[i].contiguous(), **kw)
        return np.concatenate([t.cpu().numpy().reshape(len(rx[i]), -1) for t in (r.gain, r.h_te, r.h_tm, r.parts)], 1)
    a = rows(slice(None))
    assert a[:, -1].max() > 0
    for i in {0, n_rx // 2, n_rx - 1}:
        assert np.array_equal(rows(slice(i, i + 1))[0], a[i])


@pytest.mark.parametrize("rays,n_rx", [(200, 1), (2000, 2), (20_000, 5), (60_000, 17)])
def test_refinement_parts_do_not_change_a_receiver(P, office, rays, n_rx):
    """A few key chunks and receivers are dealt in parts of a chunk; 1 024 receivers have a unit for every wavefront and
    are not. The sums of a chunk are added in key order either way."""
    rx = np.tile(scenes.office_rx(), (16, 1))
    a, r = _solve(P, office, rx[:n_rx], rays, 3)
    assert int(r.counters[P.CNT["keys"]]) > 0
    b, _ = _solve(P, office, rx, rays, 3)
    assert np.array_equal(a, b[:n_rx])


@pytest.mark.parametrize("rays,K", [(2000, 1), (2000, 3), (4000, 5), (2100, 8)])
def test_diffuse_parts_do_not_change_a_receiver(P, office, rays, K):
    """Two receivers have few (ray chunk, receiver) units, which are walked in parts and summed afterwards; 1 024
    receivers have a unit for every wavefront. The additions are the same, and so are the connections counted."""
    rx = np.tile(scenes.office_rx(), (16, 1))

    def solve(rx):
        r = P.solve(office, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, 3.5e9, rays, K=K, flags=LOS | DIFF)
        return np.concatenate([t.cpu().numpy().reshape(len(rx), -1) for t in (r.gain, r.h_te, r.h_tm, r.parts)], 1), r
    a, ra = solve(rx[:2])
    b, _ = solve(rx)
    assert a[:, -1].max() > 0 and np.array_equal(a, b[:2])
    c, rc = solve(rx[:64])
    _, rb = solve(np.tile(rx[:64], (16, 1)))
    for k in ("segments", "diffuse"):
        assert 16 * int(rc.counters[P.CNT[k]]) == int(rb.counters[P.CNT[k]])


def test_a_solve_with_few_hits_does_not_pay_for_idle_wavefronts(P, office):
    """A transmitter outside the scan: a few of its rays hit, and thousands of wavefronts have nothing to refine or
    connect. Those two stages take as long as the bounce loop (1.0 to 1.3 of it), not a queue of every wavefront at one
    counter (3.4). The nine receivers, of which none has a path, agree with a solve of one."""
    rx = scenes.office_rx()[:9]
    kw = dict(K=3, flags=LOS | SPEC | DIFF)
    ratio = []
    for _ in range(12):
        r = P.solve(office, scenes.OFFICE_MATERIALS, [100.0, 100.0, 100.0], rx, 3.5e9, 9000, K=3,
                    flags=LOS | SPEC | DIFF | P.TIMING)
        t = list(P.stage_times().values())
        ratio.append((t[3] + t[5]) / t[1])
    assert 0 < r.counter("interactions") < 100
    one = P.solve(office, scenes.OFFICE_MATERIALS, [100.0, 100.0, 100.0], rx[3:4], 3.5e9, 9000, **kw)
    assert np.array_equal(one.gain.cpu().numpy(), r.gain[3:4].cpu().numpy())
    print(ratio)
    assert min(ratio) < 2.2, ratio


def test_connections_of_one_chunk_are_dealt_over_the_chip(P, office):
    """One transmitter with 40 000 receivers, and eight equal ones with 5 000 each: the same 40 000 units of connections,
    in one chunk of records and in eight. A receiver's numbers are the same, and so are the times, bar the rest of
    the call: twice as long would mean that the units of one chunk are handed out one by one."""
    import time
    import torch
    n, rays = 40_000, 30
    rng = np.random.default_rng(n)
    at = scenes.office_rx()
    rx = np.asarray(at[rng.integers(0, len(at), n)] + rng.uniform(-0.1, 0.1, (n, 3)), np.float32)
    tx = np.repeat(np.asarray(scenes.OFFICE_TX, np.float32)[None], 8, 0)
    mats = P.materials_tensor(scenes.OFFICE_MATERIALS)
    print("[gpu-test] one chunk, many receivers", flush=True)

    def timed(f):
        r = f()
        t = []
        for _ in range(7):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return r, min(t)

    one, t1 = timed(lambda: P.solve(office, mats, scenes.OFFICE_TX, rx, 3.5e9, rays, K=2, flags=DIFF))
    eight, t8 = timed(lambda: P.solve_batch(office, mats, tx, np.full(8, rays), rx[:n // 8], 3.5e9, K=2, flags=DIFF))
    assert one.counter("diffuse") > 0
    for i in range(8):
        assert torch.equal(eight.gain[i].reshape(-1), one.gain.reshape(-1)[:n // 8])
    assert t1 < 2 * t8, (t1, t8)


@pytest.mark.parametrize("n_rx,rays,K", [(1, 30, 2), (7, 300, 3), (2000, 30, 2), (2000, 700, 1), (3100, 600, 2)])
def test_connections_of_few_chunks_do_not_change_a_receiver(P, office, n_rx, rays, K):
    """Fewer chunks than ranges of units, walked in parts and whole, with ranges that end inside a chunk: a receiver's
    numbers are those of a call with 6 500 receivers (a unit for every wavefront)."""
    rng = np.random.default_rng(rays)
    at = scenes.office_rx()
    rx = np.asarray(at[rng.integers(0, len(at), 6500)] + rng.uniform(-0.1, 0.1, (6500, 3)), np.float32)
    print("[gpu-test] few chunks %d x %d x %d" % (n_rx, rays, K), flush=True)
    full = P.solve(office, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, 3.5e9, rays, K=K, flags=DIFF)
    part = P.solve(office, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx[:n_rx], 3.5e9, rays, K=K, flags=DIFF)
    assert part.counter("diffuse") > 0 or n_rx == 1
    for a, b in ((part.gain, full.gain), (part.h_te, full.h_te), (part.parts, full.parts)):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy()[:n_rx])


@pytest.mark.parametrize("n_rx", [1, 95, 96, 97, 383, 384, 385, 767, 768, 769, 3000, 6143, 6144, 6145, 30_000])
@pytest.mark.parametrize("pol", [None, ((1.0, 0.2, -0.3), (0.1, -1.0, 0.4))])
def test_few_keys_at_many_receivers(P, room, n_rx, pol):
    """A handful of keys: units of 1 to 8 receivers, in parts, dealt or from the counter by how many there are (3 072
    wavefronts). A receiver's numbers are those of a call with 50 receivers."""
    rng = np.random.default_rng(11)
    rx = rng.uniform((0.3, 0.3, 0.3), (5.7, 3.7, 2.7), (n_rx, 3)).astype(np.float32)
    mats = scenes.box_room_materials()
    print("[gpu-test] few keys, %d receivers" % n_rx, flush=True)
    r = P.solve(room[1], mats, scenes.BOX_TX, rx, 3.5e9, 4096, K=1, flags=SPEC, pol=pol)
    assert 0 < r.counter("keys") <= 8 and r.counter("specular") > n_rx
    for lo in sorted({0, max(0, n_rx // 2 - 25), max(0, n_rx - 50)}):
        p = P.solve(room[1], mats, scenes.BOX_TX, rx[lo:lo + 50], 3.5e9, 4096, K=1, flags=SPEC, pol=pol)
        for a, b in ((r.gain, p.gain), (r.h_te, p.h_te), (r.h_tm, p.h_tm), (r.parts, p.parts)):
            assert np.array_equal(a.cpu().numpy()[lo:lo + 50], b.cpu().numpy())


def test_few_keys_at_many_receivers_do_not_wait_for_a_counter(P, room):
    """4 096 receivers of six keys take about as long as 300 (1.2 times the whole call; twice where every receiver is a unit
    of its own and all wavefronts ask one counter)."""
    import time
    import torch
    mats = P.materials_tensor(scenes.box_room_materials())
    ms = []
    for n in (300, 4096):
        rx = torch.as_tensor(np.random.default_rng(n).uniform((0.3, 0.3, 0.3), (5.7, 3.7, 2.7), (n, 3)).astype(np.float32),
                             device="cuda")
        f = lambda: P.solve(room[1], mats, scenes.BOX_TX, rx, 3.5e9, 4096, K=1, flags=SPEC)
        f()
        t = []
        for _ in range(30):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(4):
                f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        ms.append(min(t))
    assert ms[1] < 1.6 * ms[0], ms
