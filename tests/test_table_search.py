"""The rounds of the kernels' table search on the CPU: csrc/fs_common.h's own step arithmetic, compiled for the host with
signed overflow trapped, 64 probes to a round, up to the largest number of tables that the entry points take (2^31 - 1)
with offsets[t] = t and with offsets in no order."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r"""
#include "fs_common.h"
#include <cstdio>
#include <cstdlib>

template <typename Starts>
static int search(int T, Starts starts)
{
    int lo = 0, hi = T - 1;
    for (int round = 0; lo < hi; ++round) {
        const int step = fs::table_step(lo, hi);
        if (step < 1 || round > 6) { std::printf("step %d in round %d of %d tables\n", step, round, T); std::exit(1); }
        int before = 0;
        for (int lane = 0; lane < fs::kWave; ++lane) {
            const int64_t t = (int64_t)lo + (int64_t)(lane + 1) * step;
            if (t < 0) { std::printf("probe at %lld of %d tables\n", (long long)t, T); std::exit(1); }
            before += t <= hi && starts(t);
        }
        fs::table_narrow(&lo, &hi, step, before);
        if (lo < 0 || lo > hi || hi >= T) { std::printf("%d .. %d of %d tables\n", lo, hi, T); std::exit(1); }
    }
    return lo;
}

int main()
{
    const int sizes[] = {1, 2, 63, 64, 65, 66, 4096, 4097, 4098, 1 << 20, 2147483584, 2147483585, 2147483586, 2147483646, 2147483647};
    for (int T : sizes) {
        const int64_t wanted[] = {0, 1, 62, 63, 64, 65, T / 3, T / 2, T - 65, T - 64, T - 2, T - 1};
        for (int64_t i : wanted) {
            if (i < 0 || i >= T) continue;
            const int got = search(T, [&](int64_t t) { return t <= i; });
            if (got != i) { std::printf("table %d for lookup %lld of %d tables\n", got, (long long)i, T); return 1; }
        }
        search(T, [](int64_t) { return true; });
        search(T, [](int64_t t) { return (t * 2654435761u >> 7) & 1; });      // bad offsets: any answer inside [0, T)
    }
    std::printf("table search ok\n");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_rounds_stay_in_range_up_to_the_largest_number_of_tables(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    built = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
                            "-I" + os.path.join(ROCM, "include"), "-I" + os.path.join(ROOT, "include"),
                            "-I" + os.path.join(ROOT, "paper_2301_02959_amd", "csrc"), str(src), "-o", str(exe)],
                           capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "table search ok" in run.stdout, run.stdout + run.stderr
