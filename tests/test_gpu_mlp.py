"""Learned material model on the GPU: BF16 MFMA forward/backward kernels vs the
CPU reference at the kernels' rounding points, and training through the
tracer on simulator-generated channel sets.

Bars: forward outputs within 2 bf16 ulps of the activations' effect
(max |diff| <= 2e-2, mean <= 2e-3). Parameter gradients element by element:
each gradient is a sum of n products of bf16-rounded factors, and the two
sides may differ by one bf16 rounding decision in a factor (at most 2^-8 of
that term) and by the FP32 accumulation order (at most n 2^-24 of the sum of
the terms' magnitudes), so |g_gpu - g_ref| <= (2^-8 + n 2^-24) M per
element, M being that element's sum of |terms| (from the reference).
"""
import math

import numpy as np
import pytest

from oracle import mlp as R
from paper_2507_04021_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2507_04021_amd as P
    from paper_2507_04021_amd import mlp as M
    return torch, P, M


def _rows(n, n_labels, seed):
    rng = np.random.default_rng(seed)
    labels = rng.integers(0, n_labels, n).astype(np.int64)
    labels[rng.random(n) < 0.1] = 0xFFFF  # empty slots
    cosv = rng.uniform(0.0, 1.0, n).astype(np.float32)
    return labels, cosv


def _params(n_labels, seed):
    rng = np.random.default_rng(seed + 100)
    p = R.init_params(n_labels, seed=seed)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.normal(0, 0.2, size=p[k].shape)
    p["b4"][:5] = rng.normal(0, 0.3, size=5)
    return p


def _gpu_inputs(torch, labels, cosv):
    lab = torch.tensor(labels.astype(np.int32), device="cuda").to(torch.int16)
    return lab, torch.tensor(cosv, device="cuda")


@pytest.mark.parametrize("n", [1, 15, 16, 1000, 5003])
def test_mlp_forward_matches_reference(env, n):
    torch, P, M = env
    params = _params(8, 1)
    labels, cosv = _rows(n, 8, n)
    net = M.MaterialMLP(params)
    lab, cs = _gpu_inputs(torch, labels, cosv)
    out = torch.zeros(n, 8, device="cuda")
    print("[gpu-test] mlp forward n=%d" % n, flush=True)
    net.forward_rows(lab, cs, 28e9, out)
    got = out.cpu().numpy()
    live = labels != 0xFFFF
    # the kernels read FP32 master weights rounded to bf16; so does the reference
    ref = R.forward(params, labels[live], cosv[live].astype(np.float64), 28e9, precision="kernel")
    d = np.abs(got[live, :5] - ref)
    assert d.max() <= 2e-2 and d.mean() <= 2e-3, (d.max(), d.mean())
    assert np.all(got[~live] == 0) and np.all(got[:, 5:] == 0)
    assert np.all(np.hypot(got[:, 0], got[:, 1]) < 1) and np.all(np.hypot(got[:, 2], got[:, 3]) < 1)


@pytest.mark.parametrize("n", [37, 4096, 9000])
def test_mlp_backward_matches_reference(env, n):
    torch, P, M = env
    params = _params(8, 2)
    labels, cosv = _rows(n, 8, 7 + n)
    g_out = np.random.default_rng(n).normal(size=(n, 8)).astype(np.float32)
    g_out[:, 5:] = 0
    g_out[labels == 0xFFFF] = 0
    net = M.MaterialMLP(params)
    lab, cs = _gpu_inputs(torch, labels, cosv)
    print("[gpu-test] mlp backward n=%d" % n, flush=True)
    grads = net.backward_rows(lab, cs, 3.5e9, torch.tensor(g_out, device="cuda"))
    live = labels != 0xFFFF
    ref, mag = R.backward(params, labels[live], cosv[live].astype(np.float64), 3.5e9, g_out[live, :5],
                          precision="kernel", magnitudes=True)
    bound = 2.0 ** -8 + n * 2.0 ** -24
    for k, v in ref.items():
        got = grads[k].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - v) <= bound * mag[k]), (k, np.max(np.abs(got - v) / np.maximum(mag[k], 1e-300)))
        assert np.linalg.norm(got - v) <= 1e-3 * np.linalg.norm(v), k
    # padding stays structurally zero
    assert np.all(grads["W1"].cpu().numpy()[:, R.N_EMB + 2:] == 0)
    assert np.all(grads["W4"].cpu().numpy()[5:] == 0)


@pytest.mark.parametrize("n,n_labels", [(1, 1), (127, 3), (129, 17), (2049, 64), (32_769, 8), (33_000, 8), (65_537, 5)])
def test_mlp_backward_counts_every_row_once(env, n, n_labels):
    """A block takes 128 rows at a time and 256 blocks at most do, so row 32 769 starts a second round. The outputs'
    gradients are zero but for the last row, then but for the last block's first: the sum of |terms| in the bar is that
    row's alone. Then all rows, where a lost or doubled one of the small sizes shows in the norm (as above)."""
    torch, P, M = env
    params = _params(n_labels, 2)
    rng = np.random.default_rng(n)
    labels = rng.integers(0, n_labels, n).astype(np.int64)
    cosv = rng.uniform(0.0, 1.0, n).astype(np.float32)
    full = rng.normal(size=(n, 8)).astype(np.float32)
    full[:, 5:] = 0
    net = M.MaterialMLP(params)
    lab, cs = _gpu_inputs(torch, labels, cosv)
    for rows in ([n - 1], [(n - 1) // 128 * 128], range(n)):
        rows = np.asarray(rows)
        print("[gpu-test] mlp backward n=%d, %d rows with a gradient" % (n, rows.size), flush=True)
        g_out = np.zeros_like(full)
        g_out[rows] = full[rows]
        grads = net.backward_rows(lab, cs, 3.5e9, torch.tensor(g_out, device="cuda"))
        ref, mag = R.backward(params, labels[rows], cosv[rows].astype(np.float64), 3.5e9, g_out[rows, :5],
                              precision="kernel", magnitudes=True)
        for k, v in ref.items():
            got = grads[k].cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - v) <= (2.0 ** -8 + rows.size * 2.0 ** -24) * mag[k]), (rows.size, k)
            if rows.size > 1:
                assert np.linalg.norm(got - v) <= 1e-3 * np.linalg.norm(v), k


def _channel_sets(P, sg, n_sets, rays, seed):
    tx, rx = scenes.random_links(seed, n_sets, 8)
    freqs = [3.5e9 if i % 2 == 0 else 28e9 for i in range(n_sets)]
    return tx, rx, freqs


def test_mlp_training_through_the_tracer_beats_nominal_materials(env):
    """Targets from hidden per-label materials; the trained network's held-out
    dB error must be well below that of the nominal per-label Fresnel model
    (the method without the learned part)."""
    torch, P, M = env
    from paper_2507_04021_amd import diff
    s = scenes.box_room(labels="surface")
    sg = P.Scene.from_scene(s)
    truth = scenes.hidden_materials(7, 8, scatter=(0.1, 0.5))
    nominal = scenes.box_room_materials("surface", scatter=0.2)
    n_sets, rays, flags = 40, 3000, P.LOS | P.SPECULAR | P.DIFFUSE
    tx, rx, freqs = _channel_sets(P, sg, n_sets, rays, 11)
    sets = []
    print("[gpu-test] recording %d channel sets" % n_sets, flush=True)
    for i in range(n_sets):
        tgt = 10 * torch.log10(P.solve(sg, truth, tx[i], rx[i], freqs[i], rays, K=2, flags=flags).gain)
        rec = diff.record(sg, nominal, tx[i], rx[i], freqs[i], rays, K=2, flags=flags)
        sets.append((rec, freqs[i], tgt))
    train, held = sets[:32], sets[32:]

    def err_nominal(ss):
        e = []
        for rec, f, tgt in ss:
            P.tape_fresnel(rec, nominal)
            e.append(M.db_error(P.tape_forward(rec)[0], tgt))
        return float(torch.cat(e).mean())

    net = M.MaterialMLP(M.init_params(8, seed=0))
    print("[gpu-test] training", flush=True)
    hist = M.train(net, train, iters=250, batch=8, lr=5e-3)
    e_mlp = float(torch.cat([M.db_error(net.gains(rec, f), tgt) for rec, f, tgt in held]).mean())
    e_nom = err_nominal(held)
    # third comparator: the per-label Fresnel model fitted through the same tapes (gradient kernels)
    print("[gpu-test] fitting per-label materials", flush=True)
    fitted, fhist = diff.fit_per_label(train, nominal, iters=200, batch=8, lr=0.05)
    e_fit = []
    for rec, f, tgt in held:
        P.tape_fresnel(rec, fitted)
        e_fit.append(M.db_error(P.tape_forward(rec)[0], tgt))
    e_fit = float(torch.cat(e_fit).mean())
    print("[gpu-test] held-out mean |dG| dB: nominal %.3f, fitted per-label %.3f, trained network %.3f "
          "(loss %.3f -> %.3f)" % (e_nom, e_fit, e_mlp, hist[0], hist[-1]), flush=True)
    assert hist[-1] < 0.2 * hist[0]
    assert e_mlp < 0.5 * e_nom
    assert e_fit < 0.5 * e_nom and fhist[-1] < 0.2 * fhist[0]
