"""Host test of the rule that shares a batch's bytes among the waves of the
stream kernel (paper_2509_01425_amd/csrc/stream_plan.h), compiled with g++ into
a driver: the shares follow one another, cover every byte of every request
exactly once, are cut at 128-byte lines of the destination, and differ from
an equal share by less than a line at either end."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, cases):
    exe = str(tmp_path / "stream_plan_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2509_01425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "stream_plan_driver.cpp"), "-o", exe], check=True)
    text = "".join(f"{cu} {pc} {len(z)}\n" + "".join(f"{a} {b}\n" for a, b in zip(d, z))
                   for cu, pc, d, z in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


def test_shares_cover_the_batch(tmp_path):
    g = np.random.default_rng(11)
    cases = [(256, 0, [5], [0]), (256, 0, [0, 9, 700], [0, 0, 0]), (256, 0, [3], [1]),
             (256, 0, [1], [256 << 20]), (256, 0, [1], [(256 << 20) + (161 << 10)]),
             (1, 0, [77], [1 << 20]), (256, 2, [1, 1 << 40], [100 << 20, 0])]
    for _ in range(300):
        n = int(np.exp(g.uniform(0, np.log(600))))
        hi = int(np.exp(g.uniform(0, np.log(3e6))))
        z = g.integers(0, hi + 1, n) * (g.random(n) < 0.9)
        cases.append((int(g.integers(1, 305)), int(g.integers(0, 9)),
                      g.integers(0, 1 << 40, n).tolist(), z.tolist()))
    for (cu, pc, dst, size), r in zip(cases, _run(tmp_path, cases)):
        waves, s = r[0], list(zip(r[1::2], r[2::2]))
        total = int(sum(size))
        if total > (256 << 20) + len(size) * (160 << 10):
            assert waves == 0
            continue
        assert 1 <= waves <= min(4096, cu * max(pc, 1) * 4) and len(s) == waves + 1
        assert waves == 1 or (waves - 1) * 4096 < total
        assert s[-1] == (0, len(size))
        before = np.concatenate([[0], np.cumsum(size)]).astype(object)
        pos = [int(before[i] + o) for o, i in s]
        # the first share starts at byte 0 (leading empty requests aside), the
        # shares follow one another, and each cut lies inside its request
        assert pos[0] == 0 and pos[-1] == total and all(a <= b for a, b in zip(pos, pos[1:]))
        for w, (o, i) in enumerate(s[:-1]):
            assert i == len(size) or o <= size[i]
            if i < len(size) and 0 < o < size[i]:
                assert (dst[i] + o) % 128 == 0
            assert 0 <= pos[w] - total * w // waves < 128
