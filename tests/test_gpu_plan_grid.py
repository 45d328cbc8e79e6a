"""GPU: hicr_ctx_set_copy_grid between the replays of a plan.  The replays that
follow run with the new grid while earlier ones may still be in flight; bytes
and counters stay those of the oracle, and counters never fall."""
import numpy as np
import pytest

from tests.parity import expected_window, oracle_counters
from workloads import memcpy as wm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    return torch, H, wd


@pytest.mark.parametrize("n,hi", [(64, 1000), (700, 40_000), (5000, 900)])
def test_grid_set_between_replays(gpu, n, hi):
    torch, H, wd = gpu
    print("plan grid", n, hi, flush=True)
    g = np.random.default_rng(n)
    z = g.integers(0, hi, n).astype(np.uint64)
    pool = 2 * int(z.sum()) + 40 * n + 4096
    dabs, sabs = wm.layout_disjoint(g, z, pool)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    t = torch.empty(pool, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert H.hicr_slot_register(ctx, t.data_ptr(), pool)[0] == H.OK
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    d["dst_off"], d["src_off"], d["size"] = dabs, sabs, z
    assert int(np.asarray(oracle_counters(d, 1))[0][0]) == n
    want = expected_window(dabs.astype(np.int64), sabs.astype(np.int64), z.astype(np.int64), 0,
                           pool, 5)
    rc, plan, _ = H.hicr_plan_create(ctx, d)
    assert rc == H.OK, H.hicr_last_error(ctx)
    side = torch.cuda.Stream()
    done, last = 0, 0
    for grid in (0, 4, 1, 64, 2, 0, 4, 3):
        assert H.hicr_ctx_set_copy_grid(ctx, grid) == H.OK
        wd.fill(t.data_ptr(), pool, 5)
        torch.cuda.synchronize()
        for s in (0, side.cuda_stream):
            assert H.hicr_plan_launch(plan, s) == H.OK, H.hicr_last_error(ctx)
            # (what is in flight may or may not be counted yet)
            rc, sent, recv = H.hicr_slot_counters(ctx, 0)
            assert rc == H.OK and last <= sent <= (done + 1) * n and sent == recv
            last = sent
            done += 1
            # another grid while this replay may be in flight
            assert H.hicr_ctx_set_copy_grid(ctx, 5 if s else grid) == H.OK
        assert H.hicr_fence(ctx) == H.OK
        assert H.hicr_slot_counters(ctx, 0) == (H.OK, done * n, done * n)
        assert np.array_equal(t.cpu().numpy(), want), grid
    assert H.hicr_plan_destroy(plan) == H.OK
    assert H.hicr_ctx_destroy(ctx) == H.OK

