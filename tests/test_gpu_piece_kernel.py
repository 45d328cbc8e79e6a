"""GPU parity of the piece kernel (the copy of up to 4,096 requests cut into
pieces by the schedule) through the calls that still launch it at every size:
graph plans, submissions without allocation, and batches into host memory.
Every schedule class over the tiny workload, and over the alignment grid:
every (dst mod 16, src mod 16) pair with sizes around vectors, lines and the
pieces of each chunk size.  Whole pool and counters against the oracle."""
import numpy as np
import pytest

import oracle
from tests.parity import expected_window
from workloads import memcpy as wm
from workloads.content import content

pytestmark = pytest.mark.gpu

CALLS = ["graph", "noalloc", "host"]


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2509_01425_amd import hicr as H
    from workloads import device as wd
    rc, ctx = H.hicr_ctx_create(0, 0)
    assert rc == H.OK
    yield torch, H, wd, ctx
    assert H.hicr_ctx_destroy(ctx) == H.OK


def _run(env, call, d, sched):
    torch, H, wd, ctx = env
    if call != "graph":
        f = H.hicr_memcpy_batch if call == "host" else H.hicr_memcpy_batch_noalloc
        assert f(ctx, d, sched)[0] == H.OK, H.hicr_last_error(ctx)
        assert H.hicr_fence(ctx) == H.OK
        return
    rc, plan, _ = H.hicr_plan_create(ctx, d, sched, H.PLAN_GRAPH)
    assert rc == H.OK, H.hicr_last_error(ctx)
    assert H.hicr_plan_launch(plan) == H.OK
    assert H.hicr_fence(ctx) == H.OK
    assert H.hicr_plan_destroy(plan) == H.OK


@pytest.mark.parametrize("call", CALLS[:2])
@pytest.mark.parametrize("cls", range(12))
def test_tiny(env, call, cls):
    torch, H, wd, ctx = env
    bases, sizes, pool_len, descs, _ = wm.tiny(1)
    seed = 6000 + cls
    print("piece kernel tiny", call, cls, flush=True)
    pool = torch.empty(pool_len, dtype=torch.uint8, device="cuda")
    wd.fill(pool.data_ptr(), pool_len, seed)
    torch.cuda.synchronize()
    slots = np.array([H.hicr_slot_register(ctx, pool.data_ptr() + int(b), int(s))[1]
                      for b, s in zip(bases, sizes)], dtype=np.uint32)
    d = descs.copy()
    d["dst_slot"], d["src_slot"] = slots[descs["dst_slot"]], slots[descs["src_slot"]]
    _run(env, call, d, H.hicr_sched_class(cls)[1])
    host = content(seed, 0, pool_len)
    oc = oracle.Ctx()
    for b, s in zip(bases, sizes):
        oc.register(host, offset=int(b), size=int(s))
    assert oc.memcpy_batch(descs)[0] == oracle.OK
    assert np.array_equal(pool.cpu().numpy(), host)
    for k, s in enumerate(slots):
        assert H.hicr_slot_counters(ctx, int(s)) == oc.counters(k)
        assert H.hicr_slot_deregister(ctx, int(s)) == H.OK


def _grid(cls):
    """One request for every pair of alignments, its size taken in turn from
    around the edges of vectors, lines and pieces, and a few long ones."""
    from paper_2509_01425_amd import hicr as H
    chunk = H.hicr_sched_class(cls)[1].chunk_bytes
    sizes = [0, 1, 2, 15, 16, 17, 31, 127, 128, 129, 1023, 1025, 8191, 8193, 8207, 16384, 16400]
    sizes += [chunk + k for k in (-129, -1, 0, 1, 127, 144)] if chunk <= (64 << 10) else []
    g = np.random.default_rng(cls)
    reqs = [(da, sa, sizes[(16 * da + sa + 5 * cls) % len(sizes)]) for da in range(16) for sa in range(16)]
    reqs += [(3, 9, 2 * chunk + 13), (0, 0, 3 * chunk), (127, 64, chunk + 4097)]
    return [reqs[i] for i in g.permutation(len(reqs))]


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("cls", range(12))
def test_alignment_grid(env, call, cls):
    torch, H, wd, ctx = env
    print("piece kernel grid", call, cls, flush=True)
    reqs = _grid(cls)
    z = np.array([r[2] for r in reqs], np.int64)

    def place(align):  # from a line on, at the wanted distance past it
        at, cur = [], 0
        for a, n in zip(align, z):
            cur = (cur + 127) // 128 * 128 + a
            at.append(cur)
            cur += int(n) + 16
        return np.array(at, np.int64), cur + 64

    dst, d_len = place([r[0] for r in reqs])
    src, s_len = place([r[1] for r in reqs])
    d_len = (d_len + 127) // 128 * 128
    seed = 7000 + cls
    both = torch.empty(d_len + s_len, dtype=torch.uint8, device="cuda")
    wd.fill(both.data_ptr(), d_len + s_len, seed)
    torch.cuda.synchronize()
    into = both[:d_len]
    if call == "host":
        into = torch.empty(d_len, dtype=torch.uint8, pin_memory=True)
        into.copy_(both[:d_len])
    rc, a = H.hicr_slot_register(ctx, into.data_ptr(), d_len,
                                 H.MEM_HOST if call == "host" else H.MEM_HBM)
    rc2, b = H.hicr_slot_register(ctx, both.data_ptr() + d_len, s_len)
    assert rc == rc2 == H.OK, H.hicr_last_error(ctx)
    d = np.zeros(len(z), dtype=H.DESC_DTYPE)
    d["dst_slot"], d["src_slot"], d["dst_off"], d["src_off"], d["size"] = a, b, dst, src, z
    want = expected_window(dst, src + d_len, z, 0, d_len, seed)
    _run(env, call, d, H.hicr_sched_class(cls)[1])
    got = into.cpu().numpy()
    assert np.array_equal(got, want), np.nonzero(got != want)[0][:10]
    assert H.hicr_slot_counters(ctx, a) == (H.OK, 0, len(z))
    assert H.hicr_slot_counters(ctx, b) == (H.OK, len(z), 0)
    assert H.hicr_slot_deregister(ctx, a) == H.OK
    assert H.hicr_slot_deregister(ctx, b) == H.OK
