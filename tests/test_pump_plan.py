"""Host test of the rule that shares the device's workgroups among a pump's
endpoints (paper_2509_01425_amd/csrc/pump_plan.h), compiled with g++ into a
driver: what fits is exactly what four producer waves to a workgroup, one
workgroup per locking ring and one per 64 other rings fit; whatever form is
chosen stays within the device and leaves no ring without a consumer."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, cases):
    exe = str(tmp_path / "pump_plan_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2509_01425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "pump_plan_driver.cpp"), "-o", exe], check=True)
    text = "".join(f"{cap} {nl} {ni} 64 {cu} {ms} {len(w)} {' '.join(map(str, w))}\n"
                   for cap, nl, ni, w, cu, ms in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


def test_endpoint_forms(tmp_path):
    g = np.random.default_rng(3)
    cases = [c + (0, 1) for c in
             [(1536, 0, 0, []), (1536, 0, 768, []), (1536, 0, 769, []), (1536, 512, 1024, [16] * 64),
              (1536, 0, 5780, []), (1536, 0, 5781, []), (4, 5, 1, [3]), (4, 3, 3, [9, 9])]]
    for _ in range(4000):
        cap = int(g.integers(1, 1600))
        rings = int(g.integers(0, 40)) if g.random() < 0.7 else 0
        nl = sum(int(x) for x in g.integers(1, 65, rings))
        ni = int(np.exp(g.uniform(0, np.log(5 * cap + 2)))) - 1
        cases.append((cap, nl, ni, [int(x) for x in g.integers(0, 17, rings)],
                      int(g.integers(0, 300)), int(g.integers(0, 9))))
    for (cap, nl, ni, want, cu, most), r in zip(cases, _run(tmp_path, cases)):
        fits, need, lock_groups, ind_groups, units, wgs, split, share, n_team, *team = r
        assert need == (nl + ni + 3) // 4 + len(want) + (ni + 63) // 64
        assert fits == (need <= cap)
        if not fits:
            continue
        assert wgs <= cap, (cap, nl, ni, want, r)
        assert n_team == len(want) and all(1 <= t <= max(1, w) for t, w in zip(team, want))
        assert units <= ni <= 64 * units, (cap, nl, ni, want, r)
        if ind_groups:
            assert units == ni
        prod = (nl + (ni if ind_groups else (ni + 3) // 4) if lock_groups
                else ni if ind_groups else (nl + ni + 3) // 4)
        assert 1 <= share <= split <= max(1, most) and split % share == 0
        if split > 1:  # every end has as many, on compute units that nothing else uses
            assert ind_groups and ni and wgs <= cu
        assert (wgs == prod + sum(team) + (units if ind_groups else (units + 3) // 4)
                + 2 * ni * (split - 1))
    one = _run(tmp_path, cases[:6])
    assert [x[0] for x in one] == [1, 1, 1, 1, 1, 0]
    assert one[1][3] == 1 and one[2][3] == 0      # 768 streams get workgroups, 769 waves
    assert one[3][2] == 1 and one[3][8:] == [64] + [8] * 64
    few = _run(tmp_path, [(1536, 0, ni, [], 256, 8) for ni in (1, 16, 17, 32, 64, 65, 128, 129)])
    assert [x[6:8] for x in few] == [[8, 2], [8, 2], [6, 2], [4, 2], [2, 1], [1, 1], [1, 1], [1, 1]]
