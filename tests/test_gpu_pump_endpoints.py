"""The pump's endpoint forms against the CPU oracle: workgroup endpoints (few
streams), waves beside the workgroup producers of locking rings, and waves
that drain several rings each (more streams than resident waves).  Message
sizes sit at the edges of vectors, lines and chunks, on rings of an odd number
of bytes and few entries, so messages wrap at every phase."""
import numpy as np
import pytest

from tests.test_gpu_channels import _check_plan, _say, env  # noqa: F401
from workloads import channels as wc

pytestmark = pytest.mark.gpu

P, E = 10_007, 7
EDGES = np.array([0, 1, 15, 16, 17, 127, 128, 129, 1023, 3967, 4095, 4096, 4097, 8191, 8197, P],
                 dtype=np.uint64)


@pytest.mark.parametrize("mode", ["lock", "nolock"])
@pytest.mark.parametrize("n_spsc,n_mpsc,K", [(6, 1, 4), (800, 8, 4), (3300, 2, 5)])
def test_pump_endpoint_forms(env, mode, n_spsc, n_mpsc, K):  # noqa: F811
    torch, H, wd, ctx = env
    import bench
    seed, src_bytes = 77, 32 * 1024
    plan = wc.plan(n_spsc=n_spsc, n_mpsc=n_mpsc, K=K, total_msgs=17 * (n_spsc + n_mpsc * K) + 3,
                   P=P, E=E, src_bytes=src_bytes)
    g = np.random.default_rng(n_spsc)
    plan.msg_size = EDGES[g.integers(0, len(EDGES), plan.n_msgs)]
    plan.msg_src_off = np.floor(g.random(plan.n_msgs)
                                * (src_bytes - plan.msg_size.astype(np.float64) + 1)).astype(np.uint64)
    _say("pump endpoints", mode, n_spsc, n_mpsc, K)
    hmode = H.CH_MPSC_LOCK if mode == "lock" else H.CH_MPSC_NOLOCK
    rig = bench.channel_rig(torch, H, ctx, plan, hmode, seed)
    trace = torch.zeros(plan.n_msgs, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for _ in range(2):  # the second pump starts at the first one's ring positions
        rig["out"].zero_()
        torch.cuda.synchronize()
        assert H.hicr_channel_pump(ctx, rig["streams"], plan.msg_src_off, plan.msg_size,
                                   trace.data_ptr(), timeout_ns=5 * 10**9) == H.OK, \
            H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK, H.hicr_last_error(ctx)
        _check_plan(torch, H, rig, plan, seed, mode, trace)
    for ch in rig["channels"]:
        assert H.hicr_channel_destroy(ch) == H.OK


@pytest.mark.parametrize("n_spsc,n_mpsc,K,msgs", [(1, 1, 1, 600), (3, 1, 2, 300), (20, 2, 3, 41),
                                                  (60, 1, 3, 9)])
@pytest.mark.parametrize("dev", [False, True])
def test_pump_split_rings(env, n_spsc, n_mpsc, K, msgs, dev):  # noqa: F811
    """Few streams: both ends of a ring split over up to 8 workgroups, with
    groups of 1 to 16 messages, streams that end inside a group, and messages
    as large as the ring among small ones."""
    torch, H, wd, ctx = env
    import bench
    seed, src_bytes = 78, 32 * 1024
    plan = wc.plan(n_spsc=n_spsc, n_mpsc=n_mpsc, K=K, total_msgs=msgs * (n_spsc + n_mpsc * K) + 1,
                   P=P, E=E, src_bytes=src_bytes)
    g = np.random.default_rng(msgs)
    small = EDGES[:12] if n_spsc == 3 else EDGES[:6] if n_spsc == 20 else EDGES
    plan.msg_size = np.where(g.random(plan.n_msgs) < 0.97, small[g.integers(0, len(small), plan.n_msgs)],
                             P).astype(np.uint64)
    plan.msg_src_off = np.floor(g.random(plan.n_msgs)
                                * (src_bytes - plan.msg_size.astype(np.float64) + 1)).astype(np.uint64)
    _say("pump split", n_spsc, n_mpsc, K, msgs, dev)
    rig = bench.channel_rig(torch, H, ctx, plan, H.CH_MPSC_NOLOCK, seed)
    trace = torch.zeros(plan.n_msgs, dtype=torch.int32, device="cuda")
    ts = torch.zeros(2 * plan.n_msgs, dtype=torch.int64, device="cuda")
    tab = [torch.from_numpy(x.astype(np.int64)).cuda() for x in (plan.msg_src_off, plan.msg_size)]
    off, size = (tab[0].data_ptr(), tab[1].data_ptr()) if dev else (plan.msg_src_off, plan.msg_size)
    torch.cuda.synchronize()
    for _ in range(3):
        rig["out"].zero_()
        ts.zero_()
        torch.cuda.synchronize()
        kw = {"n_msgs": plan.n_msgs} if dev else {}
        assert H.hicr_channel_pump(ctx, rig["streams"], off, size, trace.data_ptr(), ts.data_ptr(),
                                   timeout_ns=5 * 10**9, **kw) == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK, H.hicr_last_error(ctx)
        _check_plan(torch, H, rig, plan, seed, "nolock", trace)
        t = ts.cpu().numpy().reshape(2, -1)
        assert (t[0] > 0).all() and (t[1] >= t[0]).all()
    for ch in rig["channels"]:
        assert H.hicr_channel_destroy(ch) == H.OK
