"""Host-API pushes whose payload several workgroups copy: messages at the edges
of a workgroup's part, up to the ring's size and across its end, pushed without
a fence between and taken out after their publication was seen, byte for byte;
and tokens, whose entries every workgroup writes some of."""
import numpy as np
import pytest

from tests.test_gpu_channels import _reg, _say, env  # noqa: F401
from workloads.content import content

pytestmark = pytest.mark.gpu

PART = 16384
SIZES = [1, PART - 1, PART, PART + 1, 2 * PART + 127, 5 * PART, 64 * PART, 64 * PART + 3]


@pytest.mark.parametrize("P", [64 * PART + 3, 3_000_017])
def test_push_large_messages(env, P):  # noqa: F811
    torch, H, wd, ctx = env
    seed, src_n, E = 91, 8 << 20, 16
    src = torch.empty(src_n, dtype=torch.uint8, device="cuda")
    wd.fill(src.data_ptr(), src_n, seed)
    ring = torch.zeros(P, dtype=torch.uint8, device="cuda")
    out = torch.zeros(src_n, dtype=torch.uint8, device="cuda")
    ent = torch.zeros(E, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    ss, rs, es, os_ = (_reg(H, ctx, t) for t in (src, ring, ent, out))
    rc, ch = H.hicr_channel_create(ctx, H.make_channel_cfg(
        H.CH_VAR, H.CH_SPSC, 1, H.CH_HOST, rs, es, capacity=P, entries=E))
    assert rc == H.OK, H.hicr_last_error(ctx)
    want = content(seed, 0, src_n)
    g = np.random.default_rng(P)
    msgs = [(int(g.integers(0, src_n - s)), s) for s in g.permutation(SIZES * 6).tolist()]
    sent = taken = 0
    while taken < len(msgs):
        while sent < len(msgs):
            rc = H.hicr_channel_push(ch, 0, ss, *msgs[sent])
            if rc == H.EAGAIN:
                break
            assert rc == H.OK, H.hicr_last_error(ctx)
            sent += 1
        rc, n, _ = H.hicr_channel_depth(ch, 0)
        assert rc == H.OK
        at = 0
        for i in range(n):
            rc, off, size, _ = H.hicr_channel_peek(ch, 0, i)
            assert rc == H.OK and size == msgs[taken + i][1]
            first = min(size, P - off)
            assert H.hicr_memcpy(ctx, os_, at, rs, off, first) == H.OK
            if size > first:
                assert H.hicr_memcpy(ctx, os_, at + first, rs, 0, size - first) == H.OK
            at += size
        if not n:
            continue
        assert H.hicr_fence(ctx) == H.OK
        got, at = out.cpu().numpy(), 0
        for i in range(n):
            off, size = msgs[taken + i]
            _say("push", P, size, off)
            assert np.array_equal(got[at:at + size], want[off:off + size]), (taken + i, size, off)
            at += size
        assert H.hicr_channel_pop(ch, 0, n) == H.OK
        taken += n
    assert H.hicr_channel_destroy(ch) == H.OK


def test_push_many_tokens(env):  # noqa: F811
    torch, H, wd, ctx = env
    T, C, seed = 48, 3000, 17
    src = torch.empty(2 * C * T, dtype=torch.uint8, device="cuda")
    wd.fill(src.data_ptr(), 2 * C * T, seed)
    ring = torch.zeros(C * T, dtype=torch.uint8, device="cuda")
    ent = torch.zeros(C, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    ss, rs, es = (_reg(H, ctx, t) for t in (src, ring, ent))
    rc, ch = H.hicr_channel_create(ctx, H.make_channel_cfg(
        H.CH_FIXED, H.CH_SPSC, 1, H.CH_HOST, rs, es, token_bytes=T, capacity=C))
    assert rc == H.OK, H.hicr_last_error(ctx)
    want = content(seed, 0, 2 * C * T)
    first = 0
    for k in (1000, C, 341, 342, 1999):  # the second fills the ring from its middle on
        _say("push tokens", k)
        ent.zero_()
        torch.cuda.synchronize()
        assert H.hicr_channel_push(ch, 0, ss, 7 * T, k) == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK
        slots = (first + np.arange(k)) % C
        assert (ent.cpu().numpy()[slots] == T).all()
        got = ring.cpu().numpy().reshape(C, T)[slots].reshape(-1)
        assert np.array_equal(got, want[7 * T:(7 + k) * T])
        assert H.hicr_channel_pop(ch, 0, k) == H.OK
        first += k
    assert H.hicr_channel_destroy(ch) == H.OK
