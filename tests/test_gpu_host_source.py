"""GPU parity of batches that read host memory, at the sizes where the number of
waves that share them changes (more of their bytes read over the host link than
from HBM, or fewer; few long requests, many short ones), as a submission and as
a plan, against the requests applied in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lo,hi,host_share", [
    (1, 4096, 4096, 1), (1, (4 << 20) + 77, (4 << 20) + 77, 1), (3, 1 << 20, 3 << 20, 1),
    (64, 60_000, 70_000, 1), (300, 0, 900, 1), (1025, 1, 20_000, 1), (4096, 1, 64, 1),
    (200, 1, 80_000, 0.5), (200, 1, 80_000, 0.1), (200, 1, 80_000, 0.9)])
def test_host_sources(n, lo, hi, host_share):
    import torch
    from paper_2509_01425_amd import hicr as H
    print("host source", n, lo, hi, host_share, flush=True)
    g = np.random.default_rng(n + lo)
    z = g.integers(lo, hi + 1, n).astype(np.int64)
    gap = g.integers(0, 40, n)
    at = np.concatenate([[0], np.cumsum(z + gap)[:-1]])
    size = int(at[-1] + z[-1]) + 64
    host = torch.empty(size, dtype=torch.uint8, pin_memory=True)
    hbm = torch.empty(size, dtype=torch.uint8, device="cuda")
    out = torch.empty(size, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    rc, o = H.hicr_slot_register(ctx, out.data_ptr(), size)
    rc, a = H.hicr_slot_register(ctx, hbm.data_ptr(), size)
    rc, b = H.hicr_slot_register(ctx, host.data_ptr(), size, H.MEM_HOST)
    assert rc == H.OK, H.hicr_last_error(ctx)
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    from_host = np.arange(n) < host_share * n
    d["dst_slot"], d["src_slot"] = o, np.where(from_host, b, a)
    d["src_off"], d["size"] = at, z
    d["dst_off"] = at + 3
    rc, plan, _ = H.hicr_plan_create(ctx, d)
    assert rc == H.OK, H.hicr_last_error(ctx)
    for k, run in enumerate([lambda: H.hicr_memcpy_batch(ctx, d)[0], lambda: H.hicr_plan_launch(plan),
                             lambda: H.hicr_memcpy_batch(ctx, d)[0]]):
        x, y = (np.random.default_rng(10 * k + j).integers(0, 256, size, dtype=np.uint8) for j in (0, 1))
        host.numpy()[:] = x
        hbm.copy_(torch.from_numpy(y))
        out.fill_(k)
        torch.cuda.synchronize()
        assert run() == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK
        want = np.full(size, k, np.uint8)
        for i in range(n):
            want[at[i] + 3:at[i] + 3 + z[i]] = (x if from_host[i] else y)[at[i]:at[i] + z[i]]
        assert np.array_equal(out.cpu().numpy(), want), k
    assert H.hicr_slot_counters(ctx, o) == (H.OK, 0, 3 * n)
    assert H.hicr_plan_destroy(plan) == H.OK
    assert H.hicr_ctx_destroy(ctx) == H.OK
