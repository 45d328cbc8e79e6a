"""GPU: the autotuner times the copy launches, not the way of the requests to
the device.  A million empty requests are 32 MB of them: over the host link
(64 GB/s in one direction at most) 24 of a request's 32 bytes alone take
393 us, while the launches over them, which move nothing, take a few tens."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LINK_BYTES_PER_S = 64e9


def test_autotune_leaves_the_upload_out():
    import torch
    from paper_2509_01425_amd import hicr as H
    n = 1 << 20
    print("autotune window", n, flush=True)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    t = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert H.hicr_slot_register(ctx, t.data_ptr(), 4096)[0] == H.OK
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    d["dst_off"] = np.arange(n) % 4096
    rc, times, _ = H.hicr_autotune(ctx, d, 3)
    assert rc == H.OK, H.hicr_last_error(ctx)
    print("times (ms)", np.round(times, 3).tolist(), flush=True)
    assert float(np.median(times)) * 1e-3 < 24 * n / LINK_BYTES_PER_S
    assert H.hicr_slot_counters(ctx, 0) == (H.OK, 0, 0)
    assert H.hicr_ctx_destroy(ctx) == H.OK
