"""The chunk schedule of launches that run several batches of one case: every
chunk runs exactly once and the grid is spread in proportion to the batches."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_spread_workgroups(tmp_path):
    exe = tmp_path / "spread_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_1109_3266_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "spread_check.cpp"), "-o", str(exe)],
                   check=True)
    rng = np.random.default_rng(5)
    cases = [(4, 4, [1]), (4, 4, [1] * 64), (5, 1, [1, 1000, 1]), (7, 2, [16, 16, 16]),
             (320, 4, [391] * 10), (320, 4, [2] * 64), (3, 8, [23, 25, 24]), (64, 1, [63]),
             (64, 1, [65])]
    for _ in range(60):
        cases.append((int(rng.integers(1, 200)), int(rng.choice([1, 2, 4, 8])),
                      rng.integers(1, rng.integers(2, 600), rng.integers(1, 65)).tolist()))
    text = "".join(f"{i} {g} {w} {' '.join(map(str, n))}\n" for i, (g, w, n) in enumerate(cases))
    out = subprocess.run([str(exe)], input=text, text=True, capture_output=True, check=True,
                         timeout=120).stdout.split("\n")
    assert out[:-1] == ["ok"] * len(cases), list(zip(cases, out))
