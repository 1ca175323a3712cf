"""Rays per work fetch (wave_rays): a given value is taken at every size, the library chooses where it is 0, and no
result depends on it."""
import ctypes

import numpy as np
import pytest

from paper_2507_04021_amd import scenes

pytestmark = pytest.mark.gpu
LOS, SPEC, DIFF = 1, 2, 4


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    import paper_2507_04021_amd as P
    P.lib()  # raises if the library is not built: no fallback
    return torch, P, P.Scene.from_scene(scenes.box_room(), width=8)


def _same(torch, P, a, b):
    for x, y in ((a.gain, b.gain), (a.h_te, b.h_te), (a.h_tm, b.h_tm), (a.parts, b.parts)):
        assert torch.equal(x, y)
    assert torch.equal(a.counters[:6], b.counters[:6])


@pytest.mark.parametrize("rays", [300, 2000, 9000, 20_000, 32_768])
def test_a_given_value_is_taken_at_every_size(env, rays):
    """Small launches that leave the choice to the library spread their rays over more wavefronts than one per 64 rays.
    A launch's wavefronts show in the workspace: each has a spill area for its stacks (8-wide nodes need one)."""
    torch, P, sg = env
    print("[gpu-test] wave_rays, %d rays" % rays, flush=True)
    assert sg.info["stack_entries"] > 23
    rx = torch.tensor([scenes.BOX_RX], dtype=torch.float32, device="cuda")
    need = {}
    for w in (0, 64, 1024):
        p = P.make_params(scenes.BOX_TX, rx, 3.5e9, rays, 1, LOS | SPEC, None, None, 0, w)
        nb = ctypes.c_size_t(0)
        assert P.lib().pcrt_solve_workspace_size(sg.handle, ctypes.byref(p), ctypes.byref(nb)) == 0
        need[w] = nb.value
    assert need[0] > need[64] >= need[1024]
    mats = scenes.box_room_materials(scatter=0.3)
    ref = P.solve(sg, mats, scenes.BOX_TX, rx, 3.5e9, rays, K=2, flags=LOS | SPEC | DIFF)
    for w in (64, 256, 1024):
        _same(torch, P, P.solve(sg, mats, scenes.BOX_TX, rx, 3.5e9, rays, K=2, flags=LOS | SPEC | DIFF, wave_rays=w), ref)


def test_fetches_from_the_counter(env):
    """More rays than the resident wavefronts are dealt at first, an odd number of them, and a batch whose
    transmitters end inside a fetch."""
    torch, P, sg = env
    print("[gpu-test] fetches of 64 to 1024 rays", flush=True)
    mats = scenes.box_room_materials(scatter=0.3)
    out = [P.solve(sg, mats, scenes.BOX_TX, [scenes.BOX_RX], 3.5e9, 600_001, K=2, flags=LOS | SPEC | DIFF, wave_rays=w)
           for w in (0, 64, 128, 256, 1024)]
    for o in out[1:]:
        _same(torch, P, o, out[0])
    tx, n = scenes.trajectory(seed=11, n=9, min_rays=1, max_rays=150_000)
    b = [P.solve_batch(sg, mats, tx, n, [scenes.BOX_RX], 3.5e9, K=2, flags=LOS | SPEC, wave_rays=w)
         for w in (0, 64, 128, 1024)]
    for o in b[1:]:
        _same(torch, P, o, b[0])
    assert b[0].counter("rays") == int(n.sum())


def test_default_of_a_solve_of_many_million_rays(env):
    """From 16 fetches of 256 rays per resident wavefront on (8 192 of them at most) the library takes 256 per fetch."""
    torch, P, sg = env
    n = 16 * 256 * 8192 + 1001
    print("[gpu-test] wave_rays, %d rays" % n, flush=True)
    mats = scenes.box_room_materials()
    a, b, c = (P.solve(sg, mats, scenes.BOX_TX, [scenes.BOX_RX], 3.5e9, n, K=1, flags=LOS | SPEC, wave_rays=w)
               for w in (0, 64, 1024))
    assert a.counter("rays") == n
    _same(torch, P, a, b)
    _same(torch, P, a, c)


def test_the_tuner_compares_the_librarys_choice_too(env, tmp_path):
    torch, P, sg = env
    s = scenes.box_room()
    choice, rows = P.autotune(s, scenes.box_room_materials(), scenes.BOX_TX, [scenes.BOX_RX], 3.5e9, 2000, K=2,
                              leaf_sizes=(2,), widths=(4,), wave_rays=(0, 64, 1024), reps=2,
                              cache_path=str(tmp_path / "tune.json"))
    assert [r["wave_rays"] for r in rows] == [0, 64, 1024] and choice["ms"] == min(r["ms"] for r in rows)
