"""GPU parity of the paths that small and many-request batches take, at the
sizes where their work split changes: single requests around a vector, a line
and a chunk, batches at the edges of a wave's 64 requests and of the 4,096
that are counted on the host, and one large enough for the host threads; each
submitted several times with no fence between (more often than there are
submission buffers) and replayed as a plan.  Whole pool and all counters
against the oracle."""
import numpy as np
import pytest

from tests.parity import expected_window, oracle_counters
from workloads import memcpy as wm

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 15, 16, 17, 111, 127, 128, 129, 1024, 4095, 4096, 4097, 8191, 12289]


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    return torch, H, wd


@pytest.mark.parametrize("n,sizes", [(1, [s]) for s in EDGES + [16384, (1 << 20) + 3]] + [
    (2, EDGES), (63, EDGES), (64, EDGES), (65, EDGES), (129, [0]), (256, [1, 17, 128, 3000]), (257, [1, 17, 128, 3000]), (255, EDGES), (300, EDGES), (4096, EDGES),
    (4097, EDGES), (20000, [1, 16, 200, 5632])])
def test_batch_sizes(gpu, n, sizes):
    torch, H, wd = gpu
    print("stream batch", n, sizes[:3], flush=True)
    g = np.random.default_rng(n * 1000 + sizes[0])
    z = np.array(sizes, np.uint64)[g.integers(0, len(sizes), n)]
    pool, n_slots, seed = 2 * int(z.sum()) + 40 * n + 4096, 7, 17 + n
    dabs, sabs = wm.layout_disjoint(g, z, pool)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    t = torch.empty(pool, dtype=torch.uint8, device="cuda")
    wd.fill(t.data_ptr(), pool, seed)
    torch.cuda.synchronize()
    # slot k reaches from k / n_slots of the pool to its end
    base = np.array([k * pool // n_slots for k in range(n_slots)], np.uint64)
    for b in base:
        assert H.hicr_slot_register(ctx, t.data_ptr() + int(b), pool - int(b))[0] == H.OK
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    for f, at in (("dst", dabs), ("src", sabs)):
        k = np.searchsorted(base, at, side="right") - 1
        k = np.maximum(k - g.integers(0, 3, n), 0)  # not only the nearest slot
        d[f + "_slot"], d[f + "_off"] = k, at - base[k]
    d["size"] = z
    want = expected_window(dabs.astype(np.int64), sabs.astype(np.int64), z.astype(np.int64), 0,
                           pool, seed)
    per_batch = oracle_counters(d, n_slots)
    done = 0

    def check(times):
        nonlocal done
        done += times
        assert H.hicr_fence(ctx) == H.OK, H.hicr_last_error(ctx)
        for k in range(n_slots):
            rc, sent, recv = H.hicr_slot_counters(ctx, k)
            assert rc == H.OK
            assert (sent, recv) == tuple(done * int(x) for x in np.asarray(per_batch)[k]), (k, done)
        assert np.array_equal(t.cpu().numpy(), want)

    assert H.hicr_memcpy_batch(ctx, d)[0] == H.OK
    check(1)
    for _ in range(6):
        assert H.hicr_memcpy_batch(ctx, d)[0] == H.OK
        for k in range(n_slots):  # what is in flight is not counted yet, or just has been
            rc, sent, recv = H.hicr_slot_counters(ctx, k)
            assert rc == H.OK and sent <= (done + 6) * int(np.asarray(per_batch)[k][0])
    check(6)
    wd.fill(t.data_ptr(), pool, seed)
    torch.cuda.synchronize()
    rc, plan, _ = H.hicr_plan_create(ctx, d)
    assert rc == H.OK, H.hicr_last_error(ctx)
    side = torch.cuda.Stream()
    for s in (0, 0, side.cuda_stream, 0):
        assert H.hicr_plan_launch(plan, s) == H.OK
    check(4)
    assert H.hicr_plan_destroy(plan) == H.OK
    if n <= 65:
        wd.fill(t.data_ptr(), pool, seed)
        torch.cuda.synchronize()
        for x in d:
            assert H.hicr_memcpy(ctx, *(int(x[f]) for f in ("dst_slot", "dst_off", "src_slot",
                                                            "src_off", "size"))) == H.OK
        check(1)
    assert H.hicr_ctx_destroy(ctx) == H.OK


@pytest.mark.parametrize("far", ["dst", "src"])
def test_small_batch_across_4_gib(gpu, far):
    """Few requests whose addresses lie 2^32 - 1, 2^32 and more bytes apart:
    kernel arguments hold them as 32-bit distances, or they go the other way."""
    torch, H, wd = gpu
    span = 1 << 32
    pool = torch.empty(span + (1 << 20), dtype=torch.uint8, device="cuda")
    small = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    small.copy_(torch.arange(1 << 20, device="cuda").remainder(251))
    for last in (span - 1, span, span + 4321):
        print("far apart", far, last, flush=True)
        rc, ctx = H.hicr_ctx_create(0, 0)
        assert rc == H.OK
        a = H.hicr_slot_register(ctx, pool.data_ptr(), pool.numel())[1]
        b = H.hicr_slot_register(ctx, small.data_ptr(), small.numel())[1]
        at, size = [0, 7777, last], 3000
        d = np.zeros(3, dtype=H.DESC_DTYPE)
        for i, o in enumerate(at):
            pool[o:o + size] = 255
            if far == "dst":
                d[i] = (a, b, o, 5000 * i + 1, size)
            else:
                pool[o:o + size] = small[5000 * i + 1:5000 * i + 1 + size]
                d[i] = (b, a, 500_000 + 5000 * i, o, size)
        torch.cuda.synchronize()
        assert H.hicr_memcpy_batch(ctx, d)[0] == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK
        for i, o in enumerate(at):
            got = (pool[o:o + size] if far == "dst"
                   else small[500_000 + 5000 * i:500_000 + 5000 * i + size])
            want = small[5000 * i + 1:5000 * i + 1 + size]
            assert torch.equal(got, want), (far, last, i)
        assert H.hicr_ctx_destroy(ctx) == H.OK
