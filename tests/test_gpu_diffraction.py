"""Single-bounce edge diffraction (Sec. II-B.3): GPU library vs the FP64
oracle, through the C ABI.

Bars: the set of (receiver, edge) pairs with a path is identical except where
an FP32 visibility walk and the FP64 test disagree at a disk rim (>= 99 % of
pairs); on pairs both keep, the complex amplitudes agree to 1e-5 relative
(both evaluate the geometry and the coefficient in FP64 from the same FP32
inputs; the GPU stores each amplitude in FP32); per-receiver sums follow.
"""
import sys

import numpy as np
import pytest

from paper_2507_04021_amd import scenes

pytestmark = pytest.mark.gpu


def step(msg):
    print("[gpu-test] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    import paper_2507_04021_amd as P
    P.lib()
    return P


@pytest.fixture(scope="module")
def small_office():
    return scenes.office(target_points=60000)


@pytest.mark.parametrize("freq,width", [(3.5e9, 4), (28e9, 2), (3.5e9, 8)])
def test_diffraction_matches_oracle(P, small_office, freq, width):
    from oracle import diffraction as dif
    sc = small_office
    edges = scenes.office_edges(sc)
    rx = scenes.office_rx()[::2]
    step("diffraction f=%g width=%d" % (freq, width))
    sg = P.Scene.from_scene(sc, leaf_size=2, width=width)
    out, amp = P.diffraction(sg, edges, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, freq, want_pairs=True)
    G, hte, htm, ref = dif.diffraction(sc, edges, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, freq)
    has_g, has_o = np.abs(amp[..., 0]) > 0, np.abs(ref[..., 0]) > 0
    assert has_o.sum() >= 50
    assert (has_g == has_o).mean() >= 0.99
    both = has_g & has_o
    err = np.abs(amp[both] - ref[both]) / np.abs(ref[both])
    assert err.max() <= 1e-5
    o = out.cpu().numpy()
    same_rx = np.all(has_g == has_o, 1)
    assert same_rx.sum() >= len(rx) // 2
    assert np.allclose(o[same_rx, 0], G[same_rx], rtol=1e-4)
    assert np.allclose(o[same_rx, 1] + 1j * o[same_rx, 2], hte[same_rx], rtol=1e-4, atol=1e-6 * np.abs(hte).max())


def test_diffraction_errors(P, small_office):
    step("diffraction errors")
    sg = P.Scene.from_scene(small_office)
    edges = scenes.office_edges(small_office)
    with pytest.raises(P.PcrtError) as e:
        P.diffraction(sg, edges, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, scenes.office_rx()[:2], -1.0)
    assert e.value.code == -1


@pytest.mark.parametrize("n_edges,n_rx", [(1, 1), (1, 65), (1, 5001), (2, 33), (3, 22), (5, 7), (32, 3), (33, 2), (64, 2),
                                          (65, 1), (160, 9)])
def test_diffraction_sums_of_a_receiver(P, small_office, n_edges, n_rx):
    """A receiver has as many lanes as there are edges, a power of two: the sums against those of the per-pair
    amplitudes (FP64 sums of at most n_edges FP32 terms)."""
    sg = P.Scene.from_scene(small_office, leaf_size=2, width=4)
    edges = scenes.office_edges(small_office)
    edges = (edges[0][-n_edges:], edges[1][-n_edges:])
    rx = np.resize(scenes.office_rx(), (n_rx, 3))
    step("diffraction sums, %d edges, %d receivers" % (n_edges, n_rx))
    out, amp = P.diffraction(sg, edges, scenes.OFFICE_MATERIALS, scenes.OFFICE_TX, rx, 3.5e9, want_pairs=True)
    amp, out = np.asarray(amp).astype(np.complex128), out.cpu().numpy()
    te, tm = amp[..., 0], amp[..., 1]
    want = np.stack([0.5 * (abs(te) ** 2 + abs(tm) ** 2).sum(1), te.real.sum(1), te.imag.sum(1), tm.real.sum(1),
                     tm.imag.sum(1)], 1)
    size = np.abs(amp).sum((1, 2))
    assert np.all(np.abs(out - want) <= 2.0 ** -52 * (n_edges + 4) * np.maximum(size, size ** 2)[:, None])


def test_diffraction_of_one_edge_takes_a_lane_per_receiver(P, small_office):
    """400 times the receivers of one edge: the chip is idle at 1 000 of them (1.2 times the time with a lane per receiver,
    15 times with a wavefront each)."""
    import torch
    sg = P.Scene.from_scene(small_office, leaf_size=2, width=4)
    edges = scenes.office_edges(small_office)
    edges = P.edges_tensor(edges[0][:1], edges[1][:1])
    mats = P.materials_tensor(scenes.OFFICE_MATERIALS)
    ms = []
    for n in (1000, 400_000):
        rx = torch.as_tensor(np.resize(scenes.office_rx(), (n, 3)).astype(np.float32), device="cuda")
        step("diffraction time, %d receivers" % n)
        P.diffraction(sg, edges, mats, scenes.OFFICE_TX, rx, 3.5e9)
        best = 1e9
        for _ in range(8):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(4):
                P.diffraction(sg, edges, mats, scenes.OFFICE_TX, rx, 3.5e9)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) / 4)
        ms.append(best)
    print(ms)
    assert ms[1] < 6 * ms[0], ms
