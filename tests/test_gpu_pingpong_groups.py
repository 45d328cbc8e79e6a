"""GPU test of the ping-pong's counter tree: workgroup counts around the one
up to which everybody polls one counter, and uneven last groups, several
sizes in one call; the pinger's and the ponger's buffers hold the message."""
import numpy as np
import pytest

from workloads.content import content

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [16, 17, 33, 250, 300])
def test_pingpong_workgroup_counts(W):
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    print("pingpong groups", W, flush=True)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    smax = (1 << 20) + 5
    bufs = [torch.zeros(smax + 16, dtype=torch.uint8, device="cuda") for _ in range(5)]
    wd.fill(bufs[0].data_ptr(), smax, 9)
    torch.cuda.synchronize()
    # 16 bytes off the start, so that stripes do not begin on lines
    slots = [H.hicr_slot_register(ctx, b.data_ptr() + 16, smax)[1] for b in bufs]
    host = content(9, 16, smax)
    for sizes in ([1, 4097, smax - 16], [40_000]):
        for b in bufs[1:]:
            b.zero_()
        torch.cuda.synchronize()
        rc, rtt = H.hicr_pingpong(ctx, *slots, sizes, 5, W)
        assert rc == H.OK, H.hicr_last_error(ctx)
        assert (rtt > 0).all() and (rtt < 10**6).all()
        n = max(sizes)
        for b in (bufs[1], bufs[4]):
            got = b.cpu().numpy()[16:]
            assert np.array_equal(got[:n], host[:n])
            assert not got[n:].any()
    assert H.hicr_ctx_destroy(ctx) == H.OK
