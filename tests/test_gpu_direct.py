"""GPU tests of the direct kernel (small scenes: every triangle tested by a
group of lanes) and of small launches whose waves hold few pixels, against the
per-pass engine and the oracle's brute force."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle
import scenegen
from paper_2312_12392_amd import rcp

pytestmark = pytest.mark.gpu

SOUP_CAM = scenegen.camera_look_at([0, 0.2, -2.5], [0, 0, 0], [0, 1, 0], 60.0)


def say(*a):
    print("[case]", *a, flush=True)


def engines_agree(s, cam, W, H, K, le, ld, mode=rcp.RCP_MODE_COLOR, z0=0.0, with_ids=True):
    a, ia = s.render(cam, W, H, K, le, ld, with_ids=with_ids, mode=mode, z0=z0)
    s.set_engine(rcp.RCP_ENGINE_PASSES)
    b, ib = s.render(cam, W, H, K, le, ld, with_ids=with_ids, mode=mode, z0=z0)
    s.set_engine(rcp.RCP_ENGINE_CHAIN)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and (not with_ids or torch.equal(ia, ib))
    return a, ia


# triangle counts around the group's 4, 16 and 64 lanes; sizes on both sides of
# the pixel counts at which the number of lanes changes (32768 and 400000)
@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 63, 64, 65, 129, 700])
def test_direct_triangle_counts(n):
    say("direct", n)
    sc = scenegen.soup_scene(seed=100 + n, n=n)
    s = rcp.Scene(sc)
    img, ids = engines_agree(s, SOUP_CAM, 61, 43, 5, 0.0, 0.05)
    o_img, o_ids = oracle.OracleScene(sc, use_bvh=False).render(SOUP_CAM, 61, 43, 5, 0.0, 0.05)
    assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()


@pytest.mark.parametrize("n,W,H", [(100, 1, 1), (100, 7, 1), (100, 181, 181), (100, 182, 181), (130, 640, 630),
                                   (100, 640, 630), (40, 640, 630), (40, 200, 150)])
@pytest.mark.parametrize("mode", [rcp.RCP_MODE_COLOR, rcp.RCP_MODE_DEPTH, rcp.RCP_MODE_NORMAL])
def test_direct_sizes_and_modes(n, W, H, mode):
    say("direct sizes", n, W, H, mode)
    s = rcp.Scene(scenegen.soup_scene(seed=7, n=n))
    engines_agree(s, SOUP_CAM, W, H, 4, 0.03, 0.1, mode, z0=1.0, with_ids=W % 2 == 1)
    s.close()


def test_direct_in_graphs_batches_and_noalloc():
    """The other entry points that take single views."""
    w = scenegen.workload("soup256")
    s = rcp.Scene(w.scene)
    img, ids = s.render(w.camera, 64, 64, 6, 0.0, 0.02)
    d = rcp.make_displacement(0.0, 0.02)
    outs = [(torch.empty_like(img), torch.empty_like(ids)) for _ in range(3)]
    rcp.rcp_render_batch(s.handle, [(w.camera, 64, 64, 6, d, *outs[0])])
    rcp.rcp_render_noalloc(s.handle, w.camera, 64, 64, 6, d, *outs[1])
    torch.cuda.synchronize()
    g = rcp.rcp_graph_create(s.handle, SOUP_CAM, 64, 64, 6, d, *outs[2])
    rcp.rcp_graph_update(g, w.camera, d)
    for _ in range(3):
        outs[2][0].zero_()
        rcp.rcp_graph_launch(g)
        torch.cuda.synchronize()
        for a, b in outs:
            assert torch.equal(a, img) and torch.equal(b, ids)
    rcp.rcp_graph_destroy(g)
    s.close()


# a wave holds 1, 2, 4 ... 64 pixels: 2 x 6144 waves at full occupancy
@pytest.mark.parametrize("W,H", [(64, 64), (160, 100), (250, 190), (400, 240), (560, 350), (800, 480), (1000, 790)])
@pytest.mark.parametrize("refill", [None, 1, 40])
def test_waves_with_few_pixels(W, H, refill):
    say("few pixels per wave", W, H, refill)
    s = rcp.Scene(scenegen.terrain_patch(seed=21, cells=90, n_boxes=40))
    if refill is not None:
        rcp.rcp_set_tuning(s.handle, refill_min=refill)
    cam = scenegen.camera_look_at([0.1, 0.4, -1.2], [0, 0.05, 0], [0, 1, 0], 60.0)
    for mode in (rcp.RCP_MODE_COLOR, rcp.RCP_MODE_NORMAL):
        engines_agree(s, cam, W, H, 4, 0.0, 0.05, mode)
    s.close()


@pytest.mark.parametrize("n,W,H", [(4097, 40, 30), (20001, 40, 30), (20001, 200, 180)])
@pytest.mark.parametrize("mode", [rcp.RCP_MODE_COLOR, rcp.RCP_MODE_NORMAL])
def test_direct_above_4096_triangles(n, W, H, mode):
    say("direct, many triangles", n, W, H, mode)
    sc = scenegen.soup_scene(seed=5, n=n)
    s = rcp.Scene(sc)
    img, ids = engines_agree(s, SOUP_CAM, W, H, 2, 0.0, 0.05, mode)
    if W * H < 2000:
        o_img, o_ids = oracle.OracleScene(sc, use_bvh=False).render(SOUP_CAM, W, H, 2, 0.0, 0.05, mode=mode)
        assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()
