"""GPU tests of the closest-hit and single-pass kernels where their launch
changes: rays in one chunk per wave, in several, and more than the lanes hold;
passes whose waves hold few pixels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle
import scenegen
from paper_2312_12392_amd import rcp

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


# 6144 waves at full occupancy: chunks of 1, 2 ... 32 rays, then several per wave
@pytest.mark.parametrize("n", [1, 63, 64, 6144, 6145, 12289, 98305, 196608, 196609, 700001])
@pytest.mark.parametrize("scene", ["soup", "terrain", "one", "empty"])
def test_trace_rays_counts(n, scene):
    say("trace rays", n, scene)
    sc = {"soup": lambda: scenegen.soup_scene(seed=2, n=90), "terrain": lambda: scenegen.terrain_patch(5, 60, 25),
          "one": lambda: scenegen.soup_scene(seed=9, n=1), "empty": scenegen.empty_scene}[scene]()
    s = rcp.Scene(sc)
    rng = np.random.default_rng(n)
    o = rng.uniform(-0.8, 0.8, (n, 3)).astype(np.float32)
    d = rng.standard_normal((n, 3)).astype(np.float32)
    t_o, t_d = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    out = [(torch.full((n,), -7.0, device="cuda"), torch.full((n,), -7, dtype=torch.int32, device="cuda"),
            torch.full((n,), -7, dtype=torch.int32, device="cuda")) for _ in range(2)]
    rcp.rcp_trace_rays(s.handle, t_o, t_d, n, *out[0])
    # the same rays in another order: every ray's result is its own
    p = torch.from_numpy(rng.permutation(n)).cuda()
    rcp.rcp_trace_rays(s.handle, t_o[p].contiguous(), t_d[p].contiguous(), n, *out[1])
    torch.cuda.synchronize()
    for a, b in zip(out[0], out[1]):
        assert torch.equal(a[p], b)
    t, i, f = (x.cpu().numpy() for x in out[0])
    assert np.all(i >= -1) and np.all((i >= 0) == np.isfinite(t)) and np.all((f == 0) | ((f == 1) & (i >= 0)))
    if sc.n_tris:
        k = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n), rng.integers(0, n, 200)]))
        ot, oi = oracle.OracleScene(sc, use_bvh=True).closest_hits(o[k], d[k], brute=True)[:2]
        assert np.array_equal(t[k], ot) and np.array_equal(i[k], oi)
    else:
        assert np.all(i == -1)
    s.close()


@pytest.mark.parametrize("W,H", [(8, 8), (100, 61), (127, 97), (350, 281), (620, 640), (1100, 800)])
@pytest.mark.parametrize("mode", [rcp.RCP_MODE_COLOR, rcp.RCP_MODE_DEPTH, rcp.RCP_MODE_NORMAL])
def test_single_passes_of_all_sizes(W, H, mode):
    """Pass k of rcp_render equals rcp_render_pass on image k - 1 and its aux."""
    say("single passes", W, H, mode)
    s = rcp.Scene(scenegen.terrain_patch(31, 80, 30))
    cam = scenegen.camera_look_at([0.1, 0.4, -1.2], [0, 0.05, 0], [0, 1, 0], 60.0)
    imgs, ids = s.render(cam, W, H, 3, 0.02, 0.06, mode=mode, z0=0.9)
    d = rcp.make_displacement(0.02, 0.06, mode, 0.9)
    prev = aux = None
    for k in range(3):
        rgb = torch.empty((H, W, 3), device="cuda")
        pid = torch.empty((H, W), dtype=torch.int32, device="cuda")
        nxt = torch.empty((H, W, 4), device="cuda")
        rcp.rcp_render_pass(s.handle, cam, W, H, d, prev, rgb, pid, prev_aux=aux, out_aux=nxt)
        torch.cuda.synchronize()
        assert torch.equal(rgb, imgs[k]) and torch.equal(pid, ids[k])
        prev, aux = rgb, nxt
    s.close()


def test_large_views_take_whole_tiles():
    """More than seven pixels per lane: waves take whole tiles and keep the rest."""
    W, H = 2112, 1400
    say("whole tiles", W, H)
    s = rcp.Scene(scenegen.terrain_patch(8, 50, 20))
    cam = scenegen.camera_look_at([0.1, 0.4, -1.2], [0, 0.05, 0], [0, 1, 0], 60.0)
    for order in (1, 0):
        rcp.rcp_set_tuning(s.handle, tile_order=order)
        a, ia = s.render(cam, W, H, 3, 0.0, 0.05)
        s.set_engine(rcp.RCP_ENGINE_PASSES)
        b, ib = s.render(cam, W, H, 3, 0.0, 0.05)
        s.set_engine(rcp.RCP_ENGINE_CHAIN)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(ia, ib)
    s.close()
