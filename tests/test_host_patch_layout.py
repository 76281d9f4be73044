"""The memory of the patch deposit: wide slots only while they take little of what is free, and
the compact ones otherwise never more than 9216 nodes for every 4096 particles."""
import itertools
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_patch_memory_is_bounded(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "patch_layout_check")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror",
                    os.path.join(ROOT, "tests", "host_check", "patch_layout_check.cpp"),
                    "-o", exe], check=True)
    cases = [(max(1, int(n ** 3 * f)), n, nbox, default, free)
             for n, f, nbox, default, free in itertools.product(
                 (8, 16, 32, 64, 128, 256, 512), (0, 0.01, 0.125, 0.375, 0.376, 0.75, 1, 4.1),
                 (1, 3, 64, 2000), (0, 1), (0, 1 << 30, 280 << 30))]
    out = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in cases) + "\n",
                         capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(cases)
    for (n_part, n, nbox, default, free), line in zip(cases, out):
        ch, slot, wide, ch0, slot0, compact, taken = map(int, line.split())
        assert slot == min(26624, n ** 3) and slot0 == min(9216, n ** 3) and ch0 == 4096
        assert wide == -(-n_part // ch) * nbox * slot * 8
        assert compact == -(-n_part // 4096) * nbox * slot0 * 8
        assert compact <= -(-n_part // 4096) * nbox * 9216 * 8
        assert bool(taken) == (wide <= 64 << 20 or (default == 1 and 8 * wide <= free))
    # a particle a node and at 3/8, 512^3, alone on the card and beside 250 GB of other data
    for n_part, free, want in ((512 ** 3, 280 << 30, 1), (512 ** 3 * 3 // 8, 280 << 30, 1),
                               (512 ** 3, 30 << 30, 0), (512 ** 3 * 3 // 8, 30 << 30, 0)):
        line = subprocess.run([exe], input=f"{n_part} 512 1 1 {free}\n", capture_output=True,
                              text=True, check=True).stdout
        assert int(line.split()[-1]) == want
