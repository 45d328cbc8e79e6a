"""Host test that the stream kernel's rule spreads short requests over its waves
(paper_2509_01425_amd/csrc/stream_plan.h), compiled with g++ into a driver: each
request is a step of its own for the wave that copies it, so no wave may be
left with a run of them while others have none.  A wave's share is bounded by
an equal share of requests and chunks, and the shares cover every byte of
every request once, in order."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stream_share") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2509_01425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "stream_share_driver.cpp"), "-o", out], check=True)
    return out


def _sizes(kind, n, g):
    if kind == "skew":
        z = np.full(n, 8)
        z[int(g.integers(0, n))] = 4 << 20
        return z
    if kind == "mixed":
        return np.floor(np.exp(g.uniform(0, np.log(64 << 10), n))).astype(np.int64)
    if kind == "edge":
        return g.choice([0, 1, 1023, 1024, 1025, 2048, 4097], n)
    return np.full(n, kind)


@pytest.mark.parametrize("n", [1, 2, 3, 64, 255, 256, 1024, 4096])
@pytest.mark.parametrize("kind", [0, 1, 16, 64, 1023, "edge", "mixed", "skew"])
def test_short_requests_are_spread(exe, n, kind):
    g = np.random.default_rng(n)
    cu = 256
    size = _sizes(kind, n, g)
    dst = g.integers(0, 1 << 40, n)
    text = f"{cu} {n}\n" + "".join(f"{a} {b}\n" for a, b in zip(dst, size))
    r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    r = [int(x) for x in r.split()]
    waves, s = r[0], list(zip(r[1::2], r[2::2]))
    assert 1 <= waves <= 4 * cu and len(s) == waves + 1 and s[0] == (0, 0) and s[-1] == (0, n)
    # at least a wave for every two short requests and for every 4 KiB, as far
    # as there are waves
    assert waves >= min(4 * cu, -(-int((size < 1024).sum()) // 2), -(-int(size.sum()) // 4096) or 1)
    before = np.concatenate([[0], np.cumsum(size)]).astype(object)
    pos = [int(before[i] + o) for o, i in s]
    assert pos == sorted(pos) and pos[-1] == int(size.sum())
    steps = 0  # of all requests: one to each, and one to every 4 KiB
    worst = 0
    for (o0, i0), (o1, i1) in zip(s, s[1:]):
        assert (i0, o0) <= (i1, o1)
        mine = 0
        for i in range(i0, min(i1 + 1, n)):
            lo, hi = (o0 if i == i0 else 0), (o1 if i == i1 else int(size[i]))
            assert 0 <= lo <= hi <= size[i]
            mine += (hi > lo) + (hi - lo) // 4096
        steps += mine
        worst = max(worst, mine)
    # (a short request counts for half a share, so a wave may hold twice an
    # equal number of steps, and one step more at either end of its share)
    assert worst <= 2 * (-(-steps // waves)) + 2, (worst, steps, waves)
