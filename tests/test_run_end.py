"""The search for a run's last chunk on the CPU: csrc/run_end.h compiled for the host, against a walk over the list.  Ascending
lists and lists in no order (a caller's own: rows that come again in later runs), whose runs have to end where their
stretch does: the list of the long runs has room for one in so many chunks, and is never written past its end."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r"""
#include "run_end.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

constexpr int64_t kChunk = 4, kLong = 3;

static void check(const std::vector<uint32_t>& keys, const char* what)
{
    const int64_t m = (int64_t)keys.size(), chunks = (m + kChunk - 1) / kChunk;
    std::vector<uint32_t> runs(chunks + 1, 0);
    for (int64_t k = 0; k < m; ++k) runs[k / kChunk + 1] += k == 0 || keys[k] != keys[k - 1];
    for (int64_t c = 0; c < chunks; ++c) runs[c + 1] += runs[c];
    int64_t long_runs = 0;
    for (int64_t c = 0; c < chunks; ++c) {
        const int64_t k0 = c * kChunk, k1 = k0 + kChunk;
        if (k1 >= m || keys[k1] != keys[k1 - 1]) continue;
        const uint32_t key = keys[k1 - 1];
        auto goes_on_into = [&](int64_t x) {                                                        // as the kernel decides
            if (x < 0 || x >= chunks) { std::printf("%s: chunk %lld of %lld\n", what, (long long)x, (long long)chunks); std::exit(1); }
            return keys[x * kChunk] == key && runs[x] == runs[c + 1];
        };
        if (k0 > 0 && keys[k0 - 1] == key && goes_on_into(c)) continue;
        const int64_t got = fs::last_chunk_of_run(c, chunks, c + 2 < chunks && goes_on_into(c + 2), goes_on_into);
        int64_t end = k1;
        while (end + 1 < m && keys[end + 1] == keys[end]) ++end;
        if (got != end / kChunk) {
            std::printf("%s: m %lld chunk %lld: %lld, not %lld\n", what, (long long)m, (long long)c, (long long)got, (long long)(end / kChunk));
            std::exit(1);
        }
        long_runs += got - c > kLong;
    }
    if (long_runs > chunks / kLong + 1) { std::printf("%s: %lld long runs in %lld chunks\n", what, (long long)long_runs, (long long)chunks); std::exit(1); }
}

int main()
{
    std::mt19937 gen(5);
    for (int m = 1; m < 400; ++m) {
        std::vector<uint32_t> keys(m);
        for (int rows : {1, 2, 3, 40}) {
            for (int stay : {0, 50, 90, 98}) {
                for (int k = 0; k < m; ++k) keys[k] = k > 0 && (int)(gen() % 100) < stay ? keys[k - 1] : gen() % rows;
                check(keys, "any order");
                std::sort(keys.begin(), keys.end());
                check(keys, "ascending");
            }
        }
        // every chunk starts with row 7, every other one is nothing else: each could be taken for a run to the list's end
        for (int k = 0; k < m; ++k) keys[k] = k % (2 * kChunk) <= kChunk ? 7 : 9;
        check(keys, "alternating");
    }
    std::printf("run ends ok\n");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_a_run_ends_with_its_stretch(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    built = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
                            "-I" + os.path.join(ROCM, "include"), "-I" + os.path.join(ROOT, "include"),
                            "-I" + os.path.join(ROOT, "paper_2301_02959_amd", "csrc"), str(src), "-o", str(exe)],
                           capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "run ends ok" in run.stdout, run.stdout + run.stderr
