"""The kernels' division of workgroup and fragment numbers by a launch's
divisors (UDiv in csrc/fs_internal.h), compiled for the host: exact for every
divisor a launch can have and numbers up to 2^24 - 1, at the multiples of the
divisor, one either side of them, and the ends of the range."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

MAIN = r"""
#include "fs_internal.h"
#include <cstdio>
int main()
{
    const int N = 1 << 24;
    long long checked = 0;
    auto check = [&](const fs::UDiv &u, int d, long long n) {
        if (n < 0 || n >= N) return true;
        ++checked;
        if (u.quo((int)n) == n / d) return true;
        std::printf("%lld / %d gives %d\n", n, d, u.quo((int)n));
        return false;
    };
    for (int d = 1; d < N; d = d < 5000 ? d + 1 : d + d / 37 + 1) {
        fs::UDiv u;
        u.set(d);
        const long long step = (N / d) / 512 + 1;
        for (long long q = 0; q * d < N; q += step)
            for (int e = -1; e <= 1; ++e)
                if (!check(u, d, q * d + e)) return 1;
        for (int e = 1; e <= 3; ++e)
            if (!check(u, d, N - e) || !check(u, d, (long long)(N - 1) / d * d - 1)) return 1;
    }
    std::printf("%lld quotients exact\n", checked);
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC) or shutil.which("g++") is None, reason="hipcc not installed")
def test_divisions_are_exact(tmp_path):
    src = tmp_path / "udiv.hip"
    src.write_text(MAIN)
    exe = str(tmp_path / "udiv")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-O2", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_1302_1700_amd", "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "quotients exact" in r.stdout, r.stdout
