"""GPU: a plan launched on a stream that the caller is capturing becomes part of
the caller's graph.  Every launch of that graph moves the plan's bytes and
raises its slots' counters once more, and the capture itself moves and counts
nothing; ordinary replays before and after count as ever.  Checked after each
of several launches of the graph, with refills and synchronisations between."""
import numpy as np
import pytest

from tests.parity import expected_window, oracle_counters
from workloads import memcpy as wm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 300, 1500, 5000])
def test_captured_plan_counts_every_launch_of_the_graph(n):
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    print("captured plan", n, flush=True)
    g = np.random.default_rng(n)
    z = g.integers(0, 6000, n).astype(np.uint64)
    pool = 2 * int(z.sum()) + 40 * n + 4096
    dabs, sabs = wm.layout_disjoint(g, z, pool)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    t = torch.empty(pool, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for _ in range(2):
        assert H.hicr_slot_register(ctx, t.data_ptr(), pool)[0] == H.OK
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    d["dst_slot"], d["src_slot"] = g.integers(0, 2, n), g.integers(0, 2, n)
    d["dst_off"], d["src_off"], d["size"] = dabs, sabs, z
    per = np.asarray(oracle_counters(d, 2)).astype(np.int64)
    rc, plan, _ = H.hicr_plan_create(ctx, d)
    assert rc == H.OK, H.hicr_last_error(ctx)
    done = 0

    def check(seed):
        for k in range(2):
            rc, sent, recv = H.hicr_slot_counters(ctx, k)
            assert (rc, sent, recv) == (H.OK, done * per[k][0], done * per[k][1]), (k, done)
        if seed:
            want = expected_window(dabs.astype(np.int64), sabs.astype(np.int64), z.astype(np.int64),
                                   0, pool, seed)
            assert np.array_equal(t.cpu().numpy(), want)

    def replay():
        nonlocal done
        wd.fill(t.data_ptr(), pool, 500 + done)
        torch.cuda.synchronize()
        assert H.hicr_plan_launch(plan) == H.OK
        assert H.hicr_fence(ctx) == H.OK
        done += 1
        check(500 + done - 1)

    replay()
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        rc = H.hicr_plan_launch(plan, s.cuda_stream)
    assert rc == H.OK, H.hicr_last_error(ctx)
    torch.cuda.synchronize()
    check(None)
    for k in range(4):
        wd.fill(t.data_ptr(), pool, 700 + k)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        done += 1
        check(700 + k)
        if k == 1:
            replay()
    graph.replay()
    graph.replay()
    torch.cuda.synchronize()
    done += 2
    check(None)
    assert H.hicr_plan_destroy(plan) == H.OK
    assert H.hicr_ctx_destroy(ctx) == H.OK


@pytest.mark.parametrize("n", [64, 5000])
def test_captured_batch_counts_every_launch_of_the_graph(n):
    """The same for a submission (whose requests stay in its staging buffer as
    long as no later submission takes it)."""
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    print("captured batch", n, flush=True)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    half = 128 * n
    t = torch.empty(2 * half, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    a = H.hicr_slot_register(ctx, t.data_ptr(), half)[1]
    b = H.hicr_slot_register(ctx, t.data_ptr() + half, half)[1]
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    d["dst_slot"], d["src_slot"], d["size"] = a, b, 100
    d["dst_off"] = d["src_off"] = 128 * np.arange(n)
    # (the submission buffers of this size exist before: a capture may not allocate)
    for _ in range(4):
        assert H.hicr_memcpy_batch(ctx, d)[0] == H.OK
    assert H.hicr_fence(ctx) == H.OK
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        rc = H.hicr_memcpy_batch(ctx, d, None, s.cuda_stream)[0]
    assert rc == H.OK, H.hicr_last_error(ctx)
    torch.cuda.synchronize()
    for k in range(3):
        assert H.hicr_slot_counters(ctx, a) == (H.OK, 0, (4 + k) * n)
        assert H.hicr_slot_counters(ctx, b) == (H.OK, (4 + k) * n, 0)
        wd.fill(t.data_ptr(), 2 * half, 80 + k)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        rows = t.cpu().numpy().reshape(2, n, 128)
        assert np.array_equal(rows[0, :, :100], rows[1, :, :100]), k
    assert H.hicr_slot_counters(ctx, a) == (H.OK, 0, 7 * n)
    assert H.hicr_ctx_destroy(ctx) == H.OK
