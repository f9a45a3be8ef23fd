"""GPU tests of the chain engine's entry lists, leaf queue and repeating
chains, against the per-pass engine (which has none of them: every ray starts
at the root and every pass is traced) and, on the small scenes, the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle
import scenegen
from paper_2312_12392_amd import rcp

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def patch_camera(eye, target=(0.0, 0.05, 0.0), fov=60.0):
    return scenegen.camera_look_at(eye, target, [0, 1, 0], fov)


def both_engines(s, cam, W, H, K, le, ld, mode=rcp.RCP_MODE_COLOR, z0=0.0, with_ids=True):
    out = []
    for e in (rcp.RCP_ENGINE_CHAIN, rcp.RCP_ENGINE_PASSES):
        s.set_engine(e)
        out.append(s.render(cam, W, H, K, le, ld, with_ids=with_ids, mode=mode, z0=z0))
    torch.cuda.synchronize()
    (a, ia), (b, ib) = out
    assert torch.equal(a, b)
    assert not with_ids or torch.equal(ia, ib)
    return a, ia


# sizes around a tile (8), a tile group (32 x 32 pixels) and the super-tiles
@pytest.mark.parametrize("W,H", [(1, 1), (31, 33), (32, 32), (65, 31), (257, 130)])
@pytest.mark.parametrize("mode,le,ld,z0", [(rcp.RCP_MODE_COLOR, 0.0, 0.05, 0.0), (rcp.RCP_MODE_COLOR, 0.3, 0.6, 0.0),
                                           (rcp.RCP_MODE_DEPTH, 0.02, 0.1, 1.0), (rcp.RCP_MODE_DEPTH, 0.5, 0.5, -3.0),
                                           (rcp.RCP_MODE_NORMAL, 0.1, 0.3, 0.0)])
def test_entry_lists_against_the_root(W, H, mode, le, ld, z0):
    """Wide displacements, a lambda beyond which no pyramid bounds the rays
    (0.6: lists without culling), eyes above, inside and under the terrain."""
    say("entry lists", W, H, mode, le, ld)
    s = rcp.Scene(scenegen.terrain_patch(seed=17, cells=40, n_boxes=30))
    for eye, target in [((0, 0.45, -1.25), (0, 0.05, 0)), ((0.1, 0.16, 0.2), (0.9, 0.1, 0.3)), ((0.3, -0.2, 0.1), (0.2, 0.6, 0.4))]:
        both_engines(s, patch_camera(eye, target), W, H, 5, le, ld, mode, z0)
    s.close()


def test_hit_beyond_the_scene_box():
    """A triangle in the plane of one pixel's ray: the test accepts it at a t
    made of rounding errors, here a quarter beyond the depth of the scene's box,
    and the pixel is displaced by so much more.  Its second ray meets a small
    triangle that no ray within the box's bound would."""
    say("hit beyond the box")
    eye = np.array([0.7027498394741156, -0.7871441872242755, 0.9608831410291954])
    cam = scenegen.camera_look_at(eye, eye + np.array([np.sin(3.8597546948284363), -0.16773908087293254,
                                                       np.cos(3.8597546948284363)]), [0, 1, 0], 60.0)
    e, f, u, r = (np.asarray(getattr(cam, n), np.float64) for n in ("eye", "forward", "up", "right"))
    a = np.array([1.2095455179417622, 1.5800046433206831, 1.8998096262026594])
    b = np.array([-2.512781526229155, 0.05199082791927978, -2.9019254816302706])
    big = e + a[:, None] * f + b[:, None] * u
    W, H, row, lam = 1, 601, 592, 0.02
    t = (1 - (2 * row + 1) / H) * float(cam.tan_half_fovy)
    p = e + 1.28 * (f + t * u + lam * 2.6299365 * r)
    small = p + 0.003 * np.array([r, -r + u, -r - u])
    rng = np.random.default_rng(0)   # the rest, off to the sides: a tree too large for the direct kernel
    c = rng.uniform(big.min(0) + 0.02, big.max(0) - 0.02, (200000, 3))
    c = c[np.abs((c - e) @ r) / np.maximum((c - e) @ f, 1e-3) > 0.15][:5000]
    verts = np.concatenate([big[None], small[None], c[:, None] + rng.uniform(-0.005, 0.005, (len(c), 3, 3))]).reshape(-1, 3)
    n = len(verts) // 3
    rgb = rng.uniform(0, 1, (n, 3))
    rgb[0] = (1.0, 0.5, 0.5)   # one to the right
    sc = scenegen.Scene(verts=verts, idx=np.arange(3 * n).reshape(n, 3), rgb=rgb)
    sc.k_a, sc.k_d = 1.0, 0.0
    o_img, o_ids = oracle.OracleScene(sc, use_bvh=True).render(cam, W, H, 3, 0.0, lam, mode=rcp.RCP_MODE_DEPTH, z0=0.0)
    assert n > 5000 and list(o_ids[:2, row, 0]) == [0, 1]   # the case is there
    s = rcp.Scene(sc, rcp.build_options(max_leaf=1))
    img, ids = both_engines(s, cam, W, H, 3, 0.0, lam, rcp.RCP_MODE_DEPTH, 0.0)
    assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()


@pytest.mark.parametrize("scale", [2.0 ** -31, 2.0 ** -33, 2.0 ** -34])
@pytest.mark.parametrize("mode", [rcp.RCP_MODE_NORMAL, rcp.RCP_MODE_DEPTH])
def test_scenes_whose_areas_are_near_the_least_float(scale, mode):
    """Squares of the triangles' normals lie among the denormals: the normals come
    out shorter and longer than 1, and displace by as much."""
    say("least areas", scale, mode)
    sc = scenegen.terrain_patch(seed=8, cells=60, n_boxes=40)
    sc.verts = (sc.verts * np.float32(scale)).astype(np.float32)
    cam = patch_camera(np.array([0.2, 0.5, -1.1]) * scale, np.array([0.0, 0.05, 0.0]) * scale)
    s = rcp.Scene(sc)
    img, ids = both_engines(s, cam, 121, 83, 4, 0.0, 0.2, mode, 0.0)
    o_img, o_ids = oracle.OracleScene(sc, use_bvh=True).render(cam, 121, 83, 4, 0.0, 0.2, mode=mode, z0=0.0)
    assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()


@pytest.mark.parametrize("fov,background", [(4.0, 0.5), (150.0, 0.5), (60.0, 3.0)])
def test_entry_lists_lens_and_background(fov, background):
    """Narrow and very wide lenses; a background above 1, which displaces by
    more than lambda (misses are not clamped by the shading table)."""
    say("entry lists lens", fov, background)
    sc = scenegen.terrain_patch(seed=3, cells=30, n_boxes=10)
    sc.background = np.full(3, background, np.float32)
    s = rcp.Scene(sc)
    cam = patch_camera((0.2, 0.5, -1.1), fov=fov)
    img, ids = both_engines(s, cam, 90, 70, 5, 0.0, 0.1)
    o_img, o_ids = oracle.OracleScene(sc, use_bvh=True).render(cam, 90, 70, 5, 0.0, 0.1)
    assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()


@pytest.mark.parametrize("max_leaf", [1, 8])
@pytest.mark.parametrize("n", [1, 2, 5, 16, 17, 300])
def test_entry_lists_of_small_trees(n, max_leaf):
    """Trees from a single leaf to more nodes than a list holds items, with
    the leaf queue's shortest and longest leaves."""
    say("entry lists, small tree", n, max_leaf)
    sc = scenegen.soup_scene(seed=n, n=n)
    s = rcp.Scene(sc, rcp.build_options(max_leaf=max_leaf))
    cam = scenegen.camera_look_at([0, 0, -2], [0, 0, 0], [0, 1, 0], 60.0)
    img, ids = both_engines(s, cam, 70, 50, 6, 0.0, 0.05)
    o_img, o_ids = oracle.OracleScene(sc, use_bvh=False).render(cam, 70, 50, 6, 0.0, 0.05)
    assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()


@pytest.mark.parametrize("K", [3, 4, 5, 7, 20])
@pytest.mark.parametrize("with_ids", [True, False])
def test_repeating_chains(K, with_ids):
    """Two and three stripes whose colours send the next ray back: many pixels
    repeat with period 2 or 3, from every pass on."""
    say("repeating chains", K, with_ids)
    rng = np.random.default_rng(5)
    n = 48
    x = np.linspace(-1.0, 1.0, n + 1)
    v, t, c = [], [], []
    for i in range(n):
        b = len(v)
        v += [[x[i], -1, 0], [x[i + 1], -1, 0], [x[i + 1], 1, 0], [x[i], 1, 0]]
        t += [[b, b + 2, b + 1], [b, b + 3, b + 2]]
        r = [(0.25, 0.75), (0.2, 0.5, 0.8)][i % 2][i // 2 % (2 + i % 2)]
        c += [[r, 0.5, 0.5], [r, 0.5, float(rng.uniform(0.4, 0.6))]]
    sc = scenegen.Scene(verts=np.array(v), idx=np.array(t), rgb=np.array(c), light=np.array([0, 0, -1.0]), name="stripes")
    s = rcp.Scene(sc)
    cam = scenegen.camera_look_at([0, 0, -1.5], [0, 0, 0], [0, 1, 0], 60.0)
    img, _ = both_engines(s, cam, 120, 40, K, 0.0, 0.06, with_ids=with_ids)
    a = img.cpu().numpy()
    if K >= 5:   # the case is there: pixels that come back after two passes without having settled
        assert np.any(np.any(a[2] != a[3], axis=-1) & np.all(a[2] == a[4], axis=-1))
    s.close()


@pytest.mark.parametrize("max_leaf", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("mode", [rcp.RCP_MODE_COLOR, rcp.RCP_MODE_DEPTH, rcp.RCP_MODE_NORMAL])
def test_leaves_of_all_sizes_in_pairs(max_leaf, mode):
    """Leaves of odd and even counts where their triangles are read two at a
    time (tests made cheap against nodes, so that leaves fill)."""
    say("pairs", max_leaf, mode)
    sc = scenegen.terrain_patch(seed=29, cells=60, n_boxes=40)
    assert sc.n_tris > 5000
    s = rcp.Scene(sc, rcp.build_options(max_leaf=max_leaf, c_isect=0.05))
    assert s.info()["leaf_hist"][max_leaf - 1] > 0
    cam = patch_camera((0.2, 0.5, -1.1))
    W, H, K = 121, 67, 4
    img, ids = both_engines(s, cam, W, H, K, 0.01, 0.05, mode, 0.9)
    o_img, o_ids = oracle.OracleScene(sc, use_bvh=True).render(cam, W, H, K, 0.01, 0.05, mode=mode, z0=0.9)
    assert np.array_equal(img.cpu().numpy(), o_img) and np.array_equal(ids.cpu().numpy(), o_ids)
    s.close()


# whole tiles around four pixels per resident lane, in the colour mode at six
# waves per SIMD of 256 compute units and in the others at five
@pytest.mark.parametrize("W", [1536, 1544])
@pytest.mark.parametrize("H,mode", [(1024, rcp.RCP_MODE_COLOR), (848, rcp.RCP_MODE_NORMAL), (856, rcp.RCP_MODE_DEPTH)])
def test_engines_agree_around_the_limit_of_few_pixels(W, H, mode):
    say("few pixels", W, H, mode)
    s = rcp.Scene(scenegen.terrain_patch(seed=8, cells=60, n_boxes=40))
    both_engines(s, patch_camera((0.2, 0.5, -1.1)), W, H, 3, 0.01, 0.05, mode, 0.9)
    s.close()


# seven pixels per resident lane are 2.75M (colour mode): from there on a wave
# takes whole tiles, where the tree's SAH cost is at most 20 per level
@pytest.mark.parametrize("W,H", [(1601, 1701), (1703, 1699)])
@pytest.mark.parametrize("scene,few_visits", [("terrain", True), ("soup", False)])
def test_engines_agree_around_the_limit_of_whole_tiles(W, H, scene, few_visits):
    say("whole tiles", W, H, scene)
    s = rcp.Scene(scenegen.terrain_patch(seed=8, cells=60, n_boxes=40) if few_visits else scenegen.soup_scene(4, 700))
    assert (s.info()["sah_cost"] <= 20.0 * s.info()["max_depth"]) == few_visits
    both_engines(s, patch_camera((0.2, 0.5, -1.1)), W, H, 2, 0.0, 0.05)
    s.close()


# the same where the rays start at the root (a view beyond the allocation-free
# area's lists), of one pass (exact counts) and of two (whole tiles), and where
# a deep tree leaves that call a smaller grid
@pytest.mark.parametrize("scene", ["terrain", "soup", "stack"])
@pytest.mark.parametrize("W,H,K", [(2600, 1900, 1), (2600, 1900, 2), (1500, 1100, 3)])
def test_whole_tiles_of_the_allocation_free_render(scene, W, H, K):
    say("whole tiles, noalloc", scene, W, H, K)
    if scene == "stack":   # a chain of triangles that halve in size: many levels
        n = 6000
        k = np.arange(n, dtype=np.float64)[:, None, None] * (40.0 / n)
        tri = np.array([[[0.0, 0.0, 0.0], [1.0, 0.1, 0.0], [0.1, 1.0, 0.3]]])
        sc = scenegen.Scene(verts=(2.0 ** (k - 40.0) * (1.0 + 0.05 * tri)).reshape(-1, 3), idx=np.arange(3 * n).reshape(n, 3),
                            rgb=np.random.default_rng(1).uniform(0, 1, (n, 3)))
    else:
        sc = scenegen.terrain_patch(seed=8, cells=60, n_boxes=40) if scene == "terrain" else scenegen.soup_scene(4, 100)
    s = rcp.Scene(sc)
    cam = patch_camera((0.2, 0.5, -1.1))
    a, ia = s.render(cam, W, H, K, 0.0, 0.05)
    b, ib = torch.empty_like(a), torch.empty_like(ia)
    rcp.rcp_render_noalloc(s.handle, cam, W, H, K, rcp.make_displacement(0.0, 0.05), b, ib)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(ia, ib)
    s.close()
