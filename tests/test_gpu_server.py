"""Continuous-batching server: every request's images equal rcp_render of
that request alone, whether it was submitted alone, in a burst, or while
other requests were running; admission respects the pool budget and the
queue capacity."""
import time

import numpy as np
import pytest
import torch

import scenegen
from paper_2312_12392_amd import rcp

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    rcp.load()


@pytest.fixture(scope="module")
def scene():
    sc = scenegen.terrain_patch(12, 40, 20)
    s = rcp.Scene(sc)
    yield s
    s.close()


def requests(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    sizes = [(64, 64), (67, 45), (1, 1), (130, 3), (96, 72), (160, 90), (33, 21)]
    for i in range(n):
        ang = rng.uniform(-0.7, 0.7)
        cam = scenegen.camera_look_at([1.4 * np.sin(ang), rng.uniform(0.3, 0.7), -1.4 * np.cos(ang)],
                                      [0, 0.05, 0], [0, 1, 0], 60.0)
        W, H = sizes[i % len(sizes)]
        K = int(rng.integers(1, 9))
        out.append((cam, W, H, K, rcp.make_displacement(0.0, float(rng.uniform(0.0, 0.1)))))
    return out


def wait_done(srv, tickets, timeout=60.0):
    t0 = time.time()
    pending = set(tickets)
    while pending:
        for t in list(pending):
            st, _ = rcp.rcp_poll(srv, t)
            assert st != rcp.RCP_REQ_FAILED, t
            if st == rcp.RCP_REQ_DONE:
                pending.discard(t)
        assert time.time() - t0 < timeout, "requests did not finish"
        time.sleep(0.001)


def check_against_alone(scene, srv, reqs, tickets):
    for (cam, W, H, K, d), t in zip(reqs, tickets):
        img = torch.empty((K, H, W, 3), device="cuda")
        ids = torch.empty((K, H, W), dtype=torch.int32, device="cuda")
        rcp.rcp_result_copy(srv, t, img, ids)
        ref_img = torch.empty_like(img)
        ref_ids = torch.empty_like(ids)
        rcp.rcp_render(scene.handle, cam, W, H, K, d, ref_img, ref_ids)
        torch.cuda.synchronize()
        assert torch.equal(img, ref_img) and torch.equal(ids, ref_ids), t
        rcp.rcp_release(srv, t)


def test_burst_equals_alone(scene):
    say("server burst")
    srv = rcp.rcp_server_create(scene.handle, 256 << 20, max_inflight=2)
    reqs = requests(24, 0)
    tickets = [rcp.rcp_submit(srv, cam, W, H, K, d, with_ids=True) for (cam, W, H, K, d) in reqs]
    wait_done(srv, tickets)
    stats = rcp.rcp_server_stats(srv)
    assert stats["launches"] < len(reqs)              # requests shared launches
    check_against_alone(scene, srv, reqs, tickets)
    assert rcp.rcp_server_stats(srv)["pool_in_use"] == 0
    rcp.rcp_server_destroy(srv)


def test_staggered_and_single_equal_alone(scene):
    say("server staggered")
    srv = rcp.rcp_server_create(scene.handle, 64 << 20, max_inflight=3)
    reqs = requests(30, 1)
    tickets = []
    for i, (cam, W, H, K, d) in enumerate(reqs):
        tickets.append(rcp.rcp_submit(srv, cam, W, H, K, d, with_ids=True))
        if i % 4 == 0:
            time.sleep(0.002)                         # arrivals while others run
    wait_done(srv, tickets)
    check_against_alone(scene, srv, reqs, tickets)
    # one request alone
    cam, W, H, K, d = reqs[4]
    t = rcp.rcp_submit(srv, cam, W, H, K, d, with_ids=True)
    wait_done(srv, [t])
    st, (ts, tb, td) = rcp.rcp_poll(srv, t)
    assert st == rcp.RCP_REQ_DONE and ts <= tb <= td
    check_against_alone(scene, srv, [reqs[4]], [t])
    rcp.rcp_server_destroy(srv)


def test_single_requests_in_cost_order_and_beyond_the_slot_order_buffer(scene):
    """A launch of one request hands its tiles out in cost order; a request
    with more tiles than a slot's order buffer holds (2^18) keeps the screen
    order.  Both equal the request rendered alone."""
    say("server single requests, small and 4200x4100")
    srv = rcp.rcp_server_create(scene.handle, 640 << 20, max_inflight=1)
    cam = scenegen.camera_look_at([0, 0.5, -1.4], [0, 0.05, 0], [0, 1, 0], 60.0)
    reqs = [(cam, 96, 64, 4, rcp.make_displacement(0.0, 0.05)),
            (cam, 4200, 4100, 1, rcp.make_displacement(0.0, 0.05))]
    for req in reqs:
        cam, W, H, K, d = req
        t = rcp.rcp_submit(srv, cam, W, H, K, d, with_ids=True)
        wait_done(srv, [t])
        check_against_alone(scene, srv, [req], [t])
    rcp.rcp_server_destroy(srv)


def test_launches_split_by_size_class(scene):
    """A launch takes the admitted requests of the oldest request's size class
    (above 2^24 pixel-passes is big): with one launch slot, a big request and
    two small ones submitted together run in two launches, the big one alone
    first; every result equals its render alone."""
    say("server size classes")
    srv = rcp.rcp_server_create(scene.handle, 512 << 20, max_inflight=1)
    cam = scenegen.camera_look_at([0.3, 0.6, -1.3], [0, 0.05, 0], [0, 1, 0], 55.0)
    d = rcp.make_displacement(0.0, 0.05)
    reqs = [(cam, 2048, 2048, 5, d), (cam, 96, 64, 3, d), (cam, 130, 70, 6, d)]
    tickets = [rcp.rcp_submit(srv, c, W, H, K, dd, with_ids=True) for (c, W, H, K, dd) in reqs]
    wait_done(srv, tickets)
    assert rcp.rcp_server_stats(srv)["launches"] == 2
    starts = [rcp.rcp_poll(srv, t)[1][1] for t in tickets]
    assert starts[0] < starts[1] == starts[2]
    check_against_alone(scene, srv, reqs, tickets)
    rcp.rcp_server_destroy(srv)


def test_mixed_modes_equal_alone(scene):
    say("server mixed modes")
    srv = rcp.rcp_server_create(scene.handle, 64 << 20, max_inflight=2)
    reqs = []
    for i, (cam, W, H, K, d) in enumerate(requests(18, 4)):
        mode = [rcp.RCP_MODE_COLOR, rcp.RCP_MODE_DEPTH, rcp.RCP_MODE_NORMAL][i % 3]
        reqs.append((cam, W, H, K, rcp.make_displacement(0.005 * (i % 2), d.lambda_dir + 0.01, mode, 1.1)))
    tickets = [rcp.rcp_submit(srv, cam, W, H, K, d, with_ids=True) for (cam, W, H, K, d) in reqs]
    wait_done(srv, tickets)
    check_against_alone(scene, srv, reqs, tickets)
    rcp.rcp_server_destroy(srv)


def test_budget_and_queue_limits(scene):
    say("server budget")
    cam, _, _, _, d = requests(1, 2)[0]
    one = 12 * 96 * 72 * 4
    pool = 2 * ((one + 255) // 256 * 256)             # two such requests fit
    srv = rcp.rcp_server_create(scene.handle, pool, max_inflight=1, queue_capacity=3)
    with pytest.raises(rcp.RcpError) as e:
        rcp.rcp_submit(srv, cam, 512, 512, 8, d)      # larger than the whole pool
    assert e.value.status == rcp.RCP_ERR_INVALID_ARGUMENT
    tickets = [rcp.rcp_submit(srv, cam, 96, 72, 4, d) for _ in range(2)]
    wait_done(srv, tickets)
    # the pool is full of finished, unreleased requests: new ones wait
    waiting = [rcp.rcp_submit(srv, cam, 96, 72, 4, d) for _ in range(3)]
    with pytest.raises(rcp.RcpError) as e:
        rcp.rcp_submit(srv, cam, 96, 72, 4, d)
    assert e.value.status == rcp.RCP_ERR_QUEUE_FULL
    time.sleep(0.05)
    assert all(rcp.rcp_poll(srv, t)[0] == rcp.RCP_REQ_QUEUED for t in waiting)
    with pytest.raises(rcp.RcpError) as e:
        rcp.rcp_result(srv, waiting[0])
    assert e.value.status == rcp.RCP_ERR_NOT_READY
    with pytest.raises(rcp.RcpError):
        rcp.rcp_release(srv, waiting[0])              # not finished yet
    for t in tickets:
        rcp.rcp_release(srv, t)                       # frees the space: two waiting ones run
    wait_done(srv, waiting[:2])
    time.sleep(0.05)
    assert rcp.rcp_poll(srv, waiting[2])[0] == rcp.RCP_REQ_QUEUED    # the pool is full again
    for t in waiting[:2]:
        assert rcp.rcp_result(srv, t)[0] != 0
        rcp.rcp_release(srv, t)
    wait_done(srv, waiting[2:])
    rcp.rcp_release(srv, waiting[2])
    assert rcp.rcp_server_stats(srv)["live"] == 0
    rcp.rcp_server_destroy(srv)


def test_more_requests_than_one_launch_holds(scene):
    """1500 tiny requests submitted at once: a launch takes at most 1024, and
    admission stops at one launch's worth waiting for a slot, so they run in
    several launches; each equals the request rendered alone."""
    rng = np.random.default_rng(21)
    reqs = []
    for i in range(1500):
        ang = rng.uniform(-0.7, 0.7)
        cam = scenegen.camera_look_at([1.4 * np.sin(ang), rng.uniform(0.3, 0.7), -1.4 * np.cos(ang)],
                                      [0, 0.05, 0], [0, 1, 0], 60.0)
        reqs.append((cam, int(rng.integers(1, 9)), int(rng.integers(1, 9)), int(rng.integers(1, 4)),
                     rcp.make_displacement(0.0, float(rng.uniform(0.0, 0.1)))))
    srv = rcp.rcp_server_create(scene.handle, 64 << 20, max_inflight=1, queue_capacity=4096)
    say("1500 requests, one launch slot")
    tickets = [rcp.rcp_submit(srv, cam, W, H, K, d, with_ids=True) for (cam, W, H, K, d) in reqs]
    wait_done(srv, tickets, timeout=120.0)
    launches = rcp.rcp_server_stats(srv)["launches"]
    assert launches >= 2, launches
    check_against_alone(scene, srv, reqs, tickets)
    assert rcp.rcp_server_stats(srv)["live"] == 0
    rcp.rcp_server_destroy(srv)


def test_destroy_with_requests_in_flight(scene):
    say("server destroy")
    srv = rcp.rcp_server_create(scene.handle, 128 << 20, max_inflight=2)
    for (cam, W, H, K, d) in requests(10, 3):
        rcp.rcp_submit(srv, cam, W, H, K, d)
    rcp.rcp_server_destroy(srv)                       # running launches finish, nothing leaks or hangs
    torch.cuda.synchronize()


@pytest.mark.parametrize("pool_gib", [3, 4])
def test_launch_of_more_groups_than_a_small_pool_holds_lists_for(pool_gib):
    """A burst of 4K requests, all but the first in one launch: ten of them have
    more tile groups than the lists of a slot at 3 GiB, fewer than at 4."""
    W, H, K, n = 3840, 2160, 2, 11
    s = rcp.Scene(scenegen.terrain_patch(8, 60, 40))
    cam = scenegen.camera_look_at([0.2, 0.5, -1.1], [0, 0.05, 0], [0, 1, 0], 60.0)
    d = rcp.make_displacement(0.0, 0.02)
    ref, _ = s.render(cam, W, H, K, 0.0, 0.02, with_ids=False)
    torch.cuda.synchronize()
    srv = rcp.rcp_server_create(s.handle, pool_gib << 30, 2, 64)
    out = torch.empty_like(ref)
    tickets = [rcp.rcp_submit(srv, cam, W, H, K, d) for _ in range(n)]
    for t in tickets:
        while rcp.rcp_poll(srv, t)[0] not in (rcp.RCP_REQ_DONE, rcp.RCP_REQ_FAILED):
            pass
        out.zero_()
        rcp.rcp_result_copy(srv, t, out, None)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        rcp.rcp_release(srv, t)
    rcp.rcp_server_destroy(srv)
    s.close()
