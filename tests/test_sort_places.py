"""Where the radix sort's passes read and write, on the CPU: csrc/radix_sort.h compiled for the host.  Every way a sort can be
given its pairs and its outputs, one to four passes, pairs side by side and (many of them) apart."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r"""
#include "radix_sort.h"
#include <cstdio>
#include <cstdlib>

static char* const base = reinterpret_cast<char*>(1ll << 40);       // addresses only: nothing is read or written

static bool overlap(const fs::SortPlace& x, const fs::SortPlace& y, int64_t m)
{
    auto ranges = [&](const fs::SortPlace& p, const char* lo[2], const char* hi[2]) {
        if (p.pairs != nullptr) { lo[0] = lo[1] = (const char*)p.pairs; hi[0] = hi[1] = lo[0] + 8 * m; return; }
        lo[0] = (const char*)p.keys; lo[1] = (const char*)p.vals; hi[0] = lo[0] + 4 * m; hi[1] = lo[1] + 4 * m;
    };
    const char *xl[2], *xh[2], *yl[2], *yh[2];
    ranges(x, xl, xh);
    ranges(y, yl, yh);
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j)
            if (xl[i] < yh[j] && yl[j] < xh[i]) return true;
    return false;
}

static void check(bool ok, const char* what, int passes, int k)
{
    if (ok) return;
    std::printf("%s: pass %d of %d\n", what, k, passes);
    std::exit(1);
}

int main()
{
    const int64_t sizes[] = {1, 1000, fs::kSortSplitFrom - 1, fs::kSortSplitFrom, fs::kSortSplitFrom + 1};
    const int64_t count = 1;
    const int64_t row = 0;
    for (int64_t m : sizes)
        for (int passes = 1; passes <= 4; ++passes)
            for (int from_rows = 0; from_rows < 2; ++from_rows)
                for (int on_device = 0; on_device < 2; ++on_device)
                    for (int out = 0; out < 4; ++out) {              // as pairs, to arrays, to the buffer that the last pass does not read,
                                                                     // to arrays that stand in for the second buffer
                        if (out == 3 && !from_rows) continue;
                        fs::SortJob job;
                        job.rows = from_rows ? &row : nullptr;
                        job.m_max = m;
                        job.m_dev = on_device ? &count : nullptr;
                        job.pairs_a = reinterpret_cast<fs::SortPair*>(base);
                        job.pairs_b = reinterpret_cast<fs::SortPair*>(base + 8 * m);
                        if (out == 3) job.pairs_b = nullptr;
                        if (out == 1 || out == 3) { job.keys_out = reinterpret_cast<uint32_t*>(base + 16 * m); job.vals_out = job.keys_out + m; }
                        if (out == 2) {
                            job.keys_out = reinterpret_cast<uint32_t*>((passes % 2 == 1) == (from_rows == 1) ? job.pairs_a : job.pairs_b);
                            job.vals_out = job.keys_out + m;
                        }
                        const fs::SortPlace start = fs::sort_place_after(job, passes, -1);
                        check(start.pairs == job.pairs_a, "the job's pairs are side by side", passes, -1);
                        for (int k = 0; k < passes; ++k) {
                            const fs::SortPlace to = fs::sort_place_after(job, passes, k);
                            check(to.pairs != nullptr || (to.keys != nullptr && to.vals != nullptr), "goes somewhere", passes, k);
                            if (k > 0 || !from_rows) check(!overlap(fs::sort_place_after(job, passes, k - 1), to, m), "reads what it writes", passes, k);
                            if (k == passes - 1 && out > 0) check(to.pairs == nullptr && to.keys == job.keys_out && to.vals == job.vals_out, "result", passes, k);
                            if (k == passes - 1 && out == 0 && (m < fs::kSortSplitFrom || on_device))
                                check(to.pairs == ((passes % 2 == 1) == (from_rows == 1) ? job.pairs_a : job.pairs_b), "result", passes, k);
                        }
                    }
    const uint32_t varying = 0;
    for (int bits = 1; bits <= 32; ++bits)                              // the digits cover the key and have a kernel each
        for (int first_bits : {0, 8, 10}) {
            if (first_bits != 0 && bits != 32) continue;
            fs::SortJob job;
            job.varying = first_bits != 0 ? &varying : nullptr;
            job.first_bits = first_bits;
            const int passes = first_bits != 0 ? 4 : fs::radix_sort_passes(bits);
            int shift = 0;
            for (int k = 0; k < passes; ++k) {
                const int digit = fs::sort_digit_bits(job, bits, passes, k, shift);
                check(digit >= (k > 0 ? fs::kSortPairsBits : 1) && digit <= fs::kSortMaxDigitBits, "digit", passes, k);
                shift += digit;
            }
            check(shift == bits, "bits", passes, bits);
        }
    std::printf("sort places ok\n");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_passes_read_what_the_one_before_wrote(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    # g++ takes the header's vector types for their elements: only addresses are looked at here
    built = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                            "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2301_02959_amd", "csrc"), str(src), "-o", str(exe)],
                           capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "sort places ok" in run.stdout, run.stdout + run.stderr
