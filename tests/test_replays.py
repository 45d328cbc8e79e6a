"""Host test of the count of a plan's ended replays
(paper_2509_01425_amd/csrc/replays.h), compiled with g++ into a driver: replays
that raise different numbers of words, in flight together, at every point
between two words."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("replays") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2509_01425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "replays_driver.cpp"), "-o", exe], check=True)

    def go(ops):
        r = subprocess.run([exe], input="\n".join(ops), capture_output=True, text=True, check=True)
        return [int(x) for x in r.stdout.split()]
    return go


def test_more_words_than_the_replay_before(run):
    # the first replay (one word) has ended; the second raises seven, and the
    # words that the first did not raise say nothing about it
    assert run(["q 1 1", "e", "r 0 1", "e", "q 7 0", "e", "r 3 2", "e"]) == [0, 1, 1, 1]
    # (known to be idle before the second)
    assert run(["q 1 1", "r 0 1", "q 7 1", "e"]) == [1]


@pytest.mark.parametrize("seed", range(40))
def test_random_replays(run, seed):
    g = np.random.default_rng(seed)
    ops, truth, seq, ended, pending = [], [], 0, 0, []
    for _ in range(60):
        if g.random() < 0.4 or not pending:
            n = int(g.choice([1, 1, 2, 7, 64]))
            ops.append(f"q {n} {int(not pending and g.random() < 0.5)}")
            seq += 1
            pending.append((seq, [int(x) for x in g.permutation(n)]))
        else:
            # the words of the oldest replay in flight go up one by one
            s, words = pending[0]
            ops.append(f"r {words.pop()} {s}")
            if not words:
                ended = s
                pending.pop(0)
        ops.append("e")
        truth.append(ended)
    got = run(ops)
    assert got == truth
