"""The learned network's walk over a grid (csrc/run.h) on the host: every run of
small ragged grids once and in order, and the runs of grids past 2^31 voxels,
whose buffers a network with few stages still fits into 288 GB."""
import os
import subprocess

import pytest

from paper_2012_04534_amd import build as B

PROGRAM = r"""
#include "run.h"
#include <cstdio>
using namespace ufss;
template <int XV> static int check(int nx, int ny, int nz, bool all) {
    const Dims d{nx, ny, nz, (int64_t)nx * ny * nz};
    const int64_t n = run_count<XV>(d), nxr = (nx + XV - 1) / XV;
    const int64_t some[] = {0, 1, n / 2, (int64_t(1) << 31) - 1, int64_t(1) << 31, (int64_t(1) << 31) + 65537, n - 1};
    for (int64_t i = 0; i < (all ? n : 7); ++i) {
        const int64_t t = all ? i : some[i];
        if (t >= n) continue;
        const Run r = run_at<XV>(d, t);
        const int64_t z = t % nz, y = t / nz / nxr, x = t / nz % nxr * XV;
        if (r.z != z || r.y != y || r.x != x || r.v != (y * nx + x) * nz + z) {
            std::printf("%d x %d x %d, runs of %d, run %lld: (%d, %d, %d) voxel %lld\n", nx, ny, nz, XV, (long long)t, r.x, r.y,
                        r.z, (long long)r.v);
            return 1;
        }
    }
    return 0;
}
template <int XV> static int checks() {
    int bad = 0;
    for (int nx : {1, 2, 3, 4, 5, 9}) bad += check<XV>(nx, 4, 7, true) + check<XV>(nx, 1, 1, true);
    return bad + check<XV>(1, 40000, 65536, false) + check<XV>(40001, 1, 65535, false) + check<XV>(300, 300, 28000, false);
}
int main() { return checks<2>() + checks<4>(); }
"""


def test_every_run_of_the_grid(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "run.hip", tmp_path / "run"
    src.write_text(PROGRAM)
    subprocess.run([B.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-I" + B.CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
