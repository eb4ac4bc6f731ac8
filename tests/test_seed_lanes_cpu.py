"""gsr_seed_triangulate takes n up to 2^31 - 1 with up to 8 neighbours; the
lanes it gives each pixel must not push the launch past the 2^32 - 1 threads
that a grid's dimension can count."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include "seed_lanes.h"
#include <stdio.h>
int main()
{
    const long long edges[] = {1, 1000, 500000, (1ll << 29) - 1, 1ll << 29, (1ll << 30) - 64, (1ll << 30) - 1, 1ll << 30,
                               (1ll << 30) + 1, (1ll << 31) - 1};
    for (long long n : edges)
        for (int k = 1; k <= 8; ++k) printf("%lld %d %d\n", n, k, gsr::seed_lanes(n, k));
    return 0;
}
"""


def test_launch_fits(tmp_path):
    src, exe = tmp_path / "lanes.cpp", tmp_path / "lanes"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2601_00705_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    rows = [tuple(map(int, line.split())) for line in
            subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines()]
    assert len(rows) == 80
    for n, k, lanes in rows:
        assert lanes in (1, 2, 4) and lanes < 2 * k
        assert -(-n * lanes // 256) * 256 < 1 << 32, (n, k, lanes)
        if n <= 1 << 29:
            assert lanes == (4 if k >= 3 else k)
