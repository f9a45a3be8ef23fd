"""GPU tests of the scene build where its launches change: cluster counts
around the merge kernels' tiles and around the size that one workgroup
finishes, deep trees, and inputs that only the device has looked at."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle
import scenegen
from paper_2312_12392_amd import rcp
from test_gpu_bvh import check_bvh

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def chain_of_sizes(n):
    """Triangles whose size and distance grow geometrically: a deep tree."""
    k = np.arange(n, dtype=np.float64)[:, None, None] * (60.0 / n)
    tri = np.array([[[0.0, 0.0, 0.0], [1.0, 0.1, 0.0], [0.1, 1.0, 0.3]]])
    v = (2.0 ** (k - 60.0) * (1.0 + 0.05 * tri)).reshape(-1, 3).astype(np.float32)
    return scenegen.Scene(verts=v, idx=np.arange(3 * n, dtype=np.uint32).reshape(-1, 3),
                          rgb=np.full((n, 3), 0.5, np.float32))


@pytest.mark.parametrize("n", [2, 5, 1023, 1024, 1025, 2048, 2049, 4095, 20481])
@pytest.mark.parametrize("make", [lambda n: scenegen.soup_scene(3, n), chain_of_sizes], ids=["soup", "deep"])
@pytest.mark.parametrize("builder", [rcp.RCP_BUILDER_PLOC, rcp.RCP_BUILDER_LBVH], ids=["ploc", "lbvh"])
@pytest.mark.parametrize("collapse", [rcp.RCP_COLLAPSE_SAH, rcp.RCP_COLLAPSE_GREEDY], ids=["sah", "greedy"])
def test_build_sizes(n, make, builder, collapse):
    say("build", n, builder, collapse)
    sc = make(n)
    opts = rcp.build_options(builder=builder, collapse=collapse)
    s, again = rcp.Scene(sc, opts), rcp.Scene(sc, opts)
    info = s.info()
    nodes, tri_ids = rcp.rcp_export_bvh(s.handle)
    check_bvh(sc, info, nodes, tri_ids)
    # leaves and cost do not depend on the order the workgroups ran in
    for key in ("n_nodes", "n_leaves", "max_depth", "sah_cost", "leaf_hist"):
        assert info[key] == again.info()[key], key
    # the tree finds what the oracle finds
    rng = np.random.default_rng(n)
    m = 200
    lo, hi = sc.verts.min(0), sc.verts.max(0)
    target = sc.verts[sc.idx[rng.integers(0, n, m)]].mean(1)
    o = rng.uniform(lo - 0.2, hi + 0.2, (m, 3)).astype(np.float32)
    d = (target - o + 1e-6).astype(np.float32)
    t, i, f = (torch.zeros(m, device="cuda"), torch.zeros(m, dtype=torch.int32, device="cuda"),
               torch.zeros(m, dtype=torch.int32, device="cuda"))
    rcp.rcp_trace_rays(s.handle, torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), m, t, i, f)
    torch.cuda.synchronize()
    ot, oi = oracle.OracleScene(sc, use_bvh=True).closest_hits(o, d, brute=True)[:2]
    assert np.array_equal(t.cpu().numpy(), ot) and np.array_equal(i.cpu().numpy(), oi)
    s.close()
    again.close()


@pytest.mark.parametrize("n", [1, 300_000])
@pytest.mark.parametrize("what,value", [("idx", 0xFFFFFFFF), ("idx", None), ("verts", np.nan), ("verts", -np.inf),
                                        ("rgb", np.inf), ("rgb", np.nan)])
def test_bad_entry_is_refused_and_named(n, what, value):
    say("bad entry", n, what, value)
    good = scenegen.soup_scene(4, n)
    arrays = {"verts": good.verts.copy(), "idx": good.idx.copy(), "rgb": good.rgb.copy()}
    arrays[what][-1, -1] = good.verts.shape[0] if value is None else value
    at = arrays[what].size - 1
    with pytest.raises(Exception) as e:
        rcp.Scene(scenegen.Scene(**arrays))
    assert str(at) in str(e.value)
    # and the next build of good arrays stands
    s = rcp.Scene(good)
    assert s.info()["n_tris"] == n
    s.close()


@pytest.mark.parametrize("what,value", [("idx", 0xFFFFFFFF), ("verts", np.nan), ("rgb", np.inf)])
@pytest.mark.parametrize("after", [0, 1, 3])
def test_bad_entry_is_the_error_when_memory_fails_too(what, value, after):
    say("bad entry without memory", what, after)
    good = scenegen.soup_scene(4, 50)
    arrays = {"verts": good.verts.copy(), "idx": good.idx.copy(), "rgb": good.rgb.copy()}
    arrays[what][-1, -1] = value
    rcp.rcp_debug_set(rcp.RCP_DEBUG_FAIL_ALLOC_AFTER, after)
    try:
        with pytest.raises(rcp.RcpError) as e:
            rcp.Scene(scenegen.Scene(**arrays))
    finally:
        rcp.rcp_debug_set(rcp.RCP_DEBUG_FAIL_ALLOC_AFTER, -1)
    assert e.value.status == rcp.RCP_ERR_INVALID_ARGUMENT and str(arrays[what].size - 1) in str(e.value)
