"""GPU: submissions without a fence between them, each of other requests than
the one before and more of them than there are submission buffers, so that a
submission that is lost, or staged over one still in flight, shows in the
bytes: every byte of every destination starts out wrong and is written by one
submission only."""
import numpy as np
import pytest

from tests.parity import expected_window, oracle_counters
from workloads import memcpy as wm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [
    [64] * 14,                                    # in the kernel's arguments
    [300] * 12,                                   # read in their pinned staging
    [1, 300, 64, 1500, 257, 4096, 2, 900, 256, 64, 1100, 3],
    [5000, 64, 9000, 300, 17_000, 1, 5001, 4096, 20_000, 700, 6000, 64],  # scanned tables too
])
@pytest.mark.parametrize("own_stream", [True, False])
def test_different_submissions_in_flight(counts, own_stream):
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    print("submission order", counts[:4], own_stream, flush=True)
    g = np.random.default_rng(sum(counts))
    n, seed = sum(counts), 8000 + len(counts)
    z = np.array([1, 16, 200, 1023, 5632], np.uint64)[g.integers(0, 5, n)]
    z = np.maximum(z, 1)
    pool = 2 * int(z.sum()) + 40 * n + 4096
    dabs, sabs = wm.layout_disjoint(g, z, pool)
    s = None if own_stream else torch.cuda.Stream()
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    t = torch.empty(pool, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for _ in range(3):
        assert H.hicr_slot_register(ctx, t.data_ptr(), pool)[0] == H.OK
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    d["dst_slot"], d["src_slot"] = g.integers(0, 3, n), g.integers(0, 3, n)
    d["dst_off"], d["src_off"], d["size"] = dabs, sabs, z
    want = expected_window(dabs.astype(np.int64), sabs.astype(np.int64), z.astype(np.int64), 0,
                           pool, seed)
    per = np.asarray(oracle_counters(d, 3)).astype(np.int64)
    parts = np.split(g.permutation(n), np.cumsum(counts)[:-1])
    for k in range(1, 4):
        wd.fill(t.data_ptr(), pool, seed)
        torch.cuda.synchronize()
        for i in g.permutation(len(parts)):
            rc, _ = H.hicr_memcpy_batch(ctx, d[parts[i]], None, 0 if s is None else s.cuda_stream)
            assert rc == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK
        got = t.cpu().numpy()
        assert np.array_equal(got, want), (k, np.nonzero(got != want)[0][:8])
        for j in range(3):
            assert H.hicr_slot_counters(ctx, j) == (H.OK, k * per[j][0], k * per[j][1])
    assert H.hicr_ctx_destroy(ctx) == H.OK
