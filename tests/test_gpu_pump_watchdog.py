"""GPU: the pump's time-out counts from the last progress a wait could see, not
from the start of the wait.  One stream alone has both ends of its ring split
over workgroups, some of which take part in large messages only: with one
large message behind many small ones they wait for nearly the whole pump,
while its counters advance all the time.  The pump must then end normally
however short its time-out is beside its run (far above any single step)."""
import numpy as np
import pytest

from tests.test_gpu_channels import _say, env  # noqa: F401
from workloads.content import content

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("large", ["last", "first and last"])
def test_split_ring_outlasts_its_timeout_while_it_moves(env, large):  # noqa: F811
    torch, H, wd, ctx = env
    n, small, big, P, E, seed = 250_001, 64, 256 << 10, 1 << 20, 64, 91
    size = np.full(n, small, np.uint64)
    size[-1] = big
    if large != "last":
        size[0] = big
    off = ((np.arange(n, dtype=np.uint64) * np.uint64(997)) % np.uint64((1 << 20) - big))
    src = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    wd.fill(src.data_ptr(), src.numel(), seed)
    out = torch.zeros(int(size.sum()), dtype=torch.uint8, device="cuda")
    ring = torch.empty(P, dtype=torch.uint8, device="cuda")
    ent = torch.zeros(E, dtype=torch.int64, device="cuda")
    ts = torch.zeros(2 * n, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    slots = [H.hicr_slot_register(ctx, t.data_ptr(), t.numel() * t.element_size())[1]
             for t in (src, out, ring, ent)]
    rc, ch = H.hicr_channel_create(ctx, H.make_channel_cfg(
        H.CH_VAR, H.CH_SPSC, 1, H.CH_DEVICE, slots[2], slots[3], capacity=P, entries=E))
    assert rc == H.OK, H.hicr_last_error(ctx)
    timeout_ns = 5_000_000
    _say("pump watchdog", large, n, timeout_ns)
    assert H.hicr_channel_pump(ctx, [(ch, 0, slots[0], slots[1], 0, n)], off, size, 0, ts.data_ptr(),
                               timeout_ns=timeout_ns) == H.OK, H.hicr_last_error(ctx)
    assert H.hicr_fence(ctx) == H.OK, H.hicr_last_error(ctx)
    t = ts.cpu().numpy()
    took = 10 * int(t.max() - t.min())  # 100 MHz
    _say("pump took (ns)", took)
    assert took > 4 * timeout_ns
    host = content(seed, 0, 1 << 20)
    want = np.concatenate([host[int(o):int(o) + int(z)] for o, z in zip(off, size)])
    assert np.array_equal(out.cpu().numpy(), want)
    assert H.hicr_channel_destroy(ch) == H.OK
    for s in slots:
        assert H.hicr_slot_deregister(ctx, s) == H.OK
