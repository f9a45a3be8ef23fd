"""GPU tests of which kernels a call launches (as the profiler names them):
rules that choose by the scene must not depend on the units of its build's
costs, nor reach past the sizes they were measured at."""
import re
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle
import scenegen
from paper_2312_12392_amd import rcp

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def launched(run):
    """Names of the kernels and runtime calls that run() makes, in order."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        torch.zeros(1, device="cuda")   # (seen in any case)
        run()
        torch.cuda.synchronize()
    names = [e.name for e in p.events()]
    if not any("elementwise" in n or "Fill" in n for n in names):
        pytest.skip("the profiler reports no kernels here")
    return [re.sub(r"^.*\(anonymous namespace\)::", "", n.split("(rcp::")[0]) if "rcp::" in n else n for n in names]


def rendered(names):
    """The rendering kernels among them: k_direct or k_chain."""
    return {m.group(0) for n in names for m in [re.match(r"k_(direct|chain)", n)] if m}


def patch_camera():
    return scenegen.camera_look_at([0.2, 0.5, -1.1], [0, 0.05, 0], [0, 1, 0], 60.0)


@pytest.mark.parametrize("scene,W,H", [("soup", 64, 64), ("soup", 640, 640), ("terrain", 120, 100)])
def test_route_does_not_depend_on_the_units_of_the_costs(scene, W, H):
    """The same tree, built with costs scaled by a power of two, takes the same
    kernels (the tree itself depends on the costs' ratio only)."""
    sc = scenegen.workload("soup256").scene if scene == "soup" else scenegen.terrain_patch(seed=8, cells=90, n_boxes=40)
    routes, trees = [], []
    for scale in (1.0, 2.0 ** -7, 2.0 ** 7):
        say("units", scene, W, H, scale)
        s = rcp.Scene(sc, rcp.build_options(c_trav=scale, c_isect=scale))
        routes.append(rendered(launched(lambda: s.render(patch_camera(), W, H, 3, 0.0, 0.02))))
        info = s.info()
        trees.append((info["n_nodes"], info["n_leaves"], info["sah_cost"] / scale))
        s.close()
    assert trees[1][:2] == trees[0][:2] == trees[2][:2] and np.allclose([t[2] for t in trees], trees[0][2], rtol=1e-6)
    assert routes[0] == routes[1] == routes[2] and len(routes[0]) == 1, routes


def with_lists(names):
    """Whether the chain kernel among them starts rays in entry lists."""
    k, = (n for n in names if n.startswith("k_chain"))
    args = re.search("<(.*)>", k).group(1).split(", ")
    return args[3 if k.startswith("k_chain_aux") else 2] == "true"


# lists where they can save levels of the tree: narrow pyramids (a spread of 0.02,
# not of 0.2, whether by the direction, a lambda that no pyramid bounds, or the
# eye), and where most of their boxes are not met anyway (soups: long chains)
@pytest.mark.parametrize("scene,W,H,K,le,ld,mode,lists", [
    ("terrain", 1920, 1080, 6, 0.0, 0.02, "color", True), ("terrain", 1920, 1080, 6, 0.0, 0.2, "color", False),
    ("terrain", 1920, 1080, 6, 0.0, 0.6, "color", False), ("terrain", 1920, 1080, 6, 0.2, 0.01, "color", False),
    ("terrain", 1280, 720, 6, 0.0, 0.2, "color", False), ("terrain", 1280, 720, 3, 0.0, 0.2, "color", True),
    ("terrain", 3840, 2160, 2, 0.0, 0.05, "color", True), ("terrain", 3840, 2160, 2, 0.0, 0.2, "color", False),
    ("terrain", 1920, 1080, 6, 0.0, 0.1, "normal", True), ("terrain", 1920, 1080, 6, 0.0, 0.4, "normal", False),
    ("soup", 3840, 2160, 1, 0.0, 0.01, "color", False), ("soup", 1920, 1080, 3, 0.0, 0.01, "color", False),
    ("soup", 1920, 1080, 6, 0.0, 0.01, "color", True), ("soup", 1280, 720, 1, 0.0, 0.01, "color", True),
    ("soup", 1920, 1080, 2, 0.0, 0.01, "normal", True)])
def test_entry_lists_where_they_pay(scene, W, H, K, le, ld, mode, lists):
    say("lists", scene, W, H, K, le, ld, mode)
    s = rcp.Scene(scenegen.terrain_patch(seed=8, cells=90, n_boxes=40) if scene == "terrain" else scenegen.soup_scene(4, 800))
    cam = patch_camera() if scene == "terrain" else scenegen.camera_look_at([0, 0.2, -2.5], [0, 0, 0], [0, 1, 0], 60.0)
    m = {"color": rcp.RCP_MODE_COLOR, "normal": rcp.RCP_MODE_NORMAL}[mode]
    d = rcp.make_displacement(le, ld, m)
    out = [(torch.empty((K, H, W, 3), device="cuda"), torch.empty((K, H, W), dtype=torch.int32, device="cuda")) for _ in range(2)]
    assert with_lists(launched(lambda: rcp.rcp_render(s.handle, cam, W, H, K, d, *out[0]))) == lists
    # a batch of one takes the same kernel, and the images are the per-pass engine's
    assert with_lists(launched(lambda: rcp.rcp_render_batch(s.handle, [(cam, W, H, K, d, *out[1])]))) == lists
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    s.set_engine(rcp.RCP_ENGINE_PASSES)
    rcp.rcp_render(s.handle, cam, W, H, K, d, *out[1])
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    s.close()


def test_batches_with_and_without_lists():
    """Views of narrow pyramids bring their lists for all; wide ones alone start
    at the root, row by row."""
    s = rcp.Scene(scenegen.terrain_patch(seed=8, cells=90, n_boxes=40))
    sizes = [(300, 200, 3), (257, 513, 2), (640, 480, 4)]
    for spreads, lists in (([0.2, 0.02, 0.3], True), ([0.2, 0.3, 0.6], False)):
        say("batch lists", spreads)
        ref = [s.render(patch_camera(), w, h, k, 0.0, ld) for (w, h, k), ld in zip(sizes, spreads)]
        out = [(torch.empty_like(a), torch.empty_like(i)) for a, i in ref]
        views = [(patch_camera(), w, h, k, rcp.make_displacement(0.0, ld), *o) for (w, h, k), ld, o in zip(sizes, spreads, out)]
        assert with_lists(launched(lambda: rcp.rcp_render_batch(s.handle, views))) == lists
        for (a, i), (b, j) in zip(ref, out):
            assert torch.equal(a, b) and torch.equal(i, j)
    s.close()


# soups of large triangles, where the direct kernel's share ends: K passes of
# the tree take 0.7e9 tests' time each at 4096 triangles, and nothing was
# measured beyond 262,144
@pytest.mark.parametrize("n,W,H,K,direct", [(4096, 400, 300, 1, True), (4096, 720, 480, 1, False), (4096, 720, 480, 3, True),
                                            (16384, 512, 512, 1, False), (262144, 32, 32, 1, True), (262145, 32, 32, 1, False)])
def test_direct_kernel_only_where_it_was_measured_faster(n, W, H, K, direct):
    say("direct limit", n, W, H, K)
    s = rcp.Scene(scenegen.soup_scene(seed=3, n=n))
    cam = scenegen.camera_look_at([0, 0.2, -2.5], [0, 0, 0], [0, 1, 0], 60.0)
    assert rendered(launched(lambda: s.render(cam, W, H, K, 0.0, 0.02))) == {"k_direct" if direct else "k_chain"}
    s.close()


def test_server_launches_start_after_a_long_direct_launch():
    """A direct launch that keeps the chip busy is not run beside others; every
    request's images are those of rcp_render."""
    say("server beside a direct launch")
    s = rcp.Scene(scenegen.soup_scene(seed=12, n=4000))
    cam = scenegen.camera_look_at([0, 0.2, -2.5], [0, 0, 0], [0, 1, 0], 60.0)
    d = rcp.make_displacement(0.0, 0.02)
    sizes = [(512, 512, 8), (64, 64, 1), (1280, 720, 1)]   # the first one runs for milliseconds
    ref = [s.render(cam, w, h, k, 0.0, 0.02) for w, h, k in sizes]
    srv = rcp.rcp_server_create(s.handle, 1 << 30, max_inflight=3)
    for _ in range(5):
        tickets, done = [], []
        for w, h, k in sizes:
            tickets.append(rcp.rcp_submit(srv, cam, w, h, k, d, with_ids=True))
            time.sleep(0.0003)   # a launch each
        for t, (img, ids) in zip(tickets, ref):
            while (p := rcp.rcp_poll(srv, t))[0] not in (rcp.RCP_REQ_DONE, rcp.RCP_REQ_FAILED):
                pass
            done.append(p[1][2])
            a, b = torch.empty_like(img), torch.empty_like(ids)
            rcp.rcp_result_copy(srv, t, a, b)
            torch.cuda.synchronize()
            assert torch.equal(a, img) and torch.equal(b, ids)
            rcp.rcp_release(srv, t)
        assert done[0] <= min(done[1:]), done
    rcp.rcp_server_destroy(srv)
    s.close()


def test_views_of_crossing_needs_share_one_workspace():
    """1290 x 720 takes more tiles (padded), 1024 x 1024 more groups: rendered in
    turn, only the first two frames allocate."""
    s = rcp.Scene(scenegen.terrain_patch(seed=8, cells=90, n_boxes=40))
    sizes = [(1290, 720), (1024, 1024)]
    out = [torch.empty((2, h, w, 3), device="cuda") for w, h in sizes]
    d = rcp.make_displacement(0.0, 0.02)

    def both():
        for (w, h), o in zip(sizes, out):
            rcp.rcp_render(s.handle, patch_camera(), w, h, 2, d, o, None)

    both()
    both()
    say("alternating views")
    names = launched(lambda: [both() for _ in range(3)])
    assert sum(n.startswith("k_chain") for n in names) == 6
    assert not any("Malloc" in n for n in names if n != "hipStreamIsCapturing"), names
    s.close()


def test_views_beyond_the_most_lists():
    """Views one pixel wide under tiles 64 wide have a list per four pixels: from
    2^20 lists on (the bound of batches and, now, of single renders) rays start
    at the root.  The same images come from tiles 8 wide."""
    s = rcp.Scene(scenegen.terrain_patch(seed=8, cells=90, n_boxes=40))
    cam = scenegen.camera_look_at([0.2, 0.5, -1.1], [0, 0.05, 0], [0, 1, 0], 100.0)
    W, H, K = 1, (1 << 22) + 8, 2
    d = rcp.make_displacement(0.0, 0.02)
    out = [(torch.empty((K, H, W, 3), device="cuda"), torch.empty((K, H, W), dtype=torch.int32, device="cuda")) for _ in range(3)]
    say("beyond the most lists")
    rcp.rcp_render(s.handle, cam, W, H, K, d, *out[0])
    rcp.rcp_set_tuning(s.handle, tile_log2w=6)
    assert not with_lists(launched(lambda: rcp.rcp_render(s.handle, cam, W, H, K, d, *out[1])))
    small = (torch.empty((1, 40, 30, 3), device="cuda"), None)
    views = [(cam, W, H, K, d, *out[2]), (cam, 30, 40, 1, d, *small)]
    assert not with_lists(launched(lambda: rcp.rcp_render_batch(s.handle, views)))
    for a, b in out[1:]:
        assert torch.equal(a, out[0][0]) and torch.equal(b, out[0][1])
    s.close()
