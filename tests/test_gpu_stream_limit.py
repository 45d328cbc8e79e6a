"""GPU parity of batches around the size up to which a schedule of 4 KiB pieces
leaves them to the stream kernel (160 MiB and 160 KiB a request), as a
submission and as a plan, under a class of 4 KiB pieces and one of 64 KiB."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cls", [0, 4])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_around_the_limit_of_small_pieces(cls, over):
    import torch
    from paper_2509_01425_amd import hicr as H
    n = 5
    total = (160 << 20) + n * (160 << 10) + over
    print("stream limit", cls, over, flush=True)
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    half = total + 64 * n
    t = torch.empty(2 * half, dtype=torch.uint8, device="cuda")
    src = (torch.arange(half, device="cuda", dtype=torch.int64) * 2654435761 >> 13).to(torch.uint8)
    a = H.hicr_slot_register(ctx, t.data_ptr(), half)[1]
    b = H.hicr_slot_register(ctx, t.data_ptr() + half, half)[1]
    size = np.array([1, 4097, 30 << 20, 77], np.int64)
    size = np.append(size, total - size.sum())
    d = np.zeros(n, dtype=H.DESC_DTYPE)
    d["dst_slot"], d["src_slot"], d["size"] = a, b, size
    at = np.concatenate([[0], np.cumsum(size + 13)[:-1]])
    d["dst_off"], d["src_off"] = at + 3, at + 8
    want = torch.full((half,), 7, dtype=torch.uint8, device="cuda")
    for o, z in zip(at, size):
        want[o + 3:o + 3 + z] = src[o + 8:o + 8 + z]
    rc, plan, _ = H.hicr_plan_create(ctx, d, H.hicr_sched_class(cls)[1])
    assert rc == H.OK, H.hicr_last_error(ctx)
    for run in (lambda: H.hicr_memcpy_batch(ctx, d, H.hicr_sched_class(cls)[1])[0],
                lambda: H.hicr_plan_launch(plan)):
        t[:half] = 7
        t[half:] = src
        torch.cuda.synchronize()
        assert run() == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK
        assert torch.equal(t[:half], want) and torch.equal(t[half:], src)
    assert H.hicr_slot_counters(ctx, a) == (H.OK, 0, 2 * n)
    assert H.hicr_plan_destroy(plan) == H.OK
    assert H.hicr_ctx_destroy(ctx) == H.OK
