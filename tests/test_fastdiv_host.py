"""Division by a launch constant (csrc/znn_internal.h), on the CPU: exact for every dividend and divisor that a kernel may be given."""
import os
import subprocess

from paper_1510_06706_amd import build

SOURCE = r"""
#include <cstdio>
#include "znn_internal.h"
int main()
{
    const unsigned divisors[] = {1, 2, 3, 5, 7, 12, 64, 1000, 65535, 65536, 65537, 75001, 150000, 500000, 1u << 20, 123456789u, 1u << 30};
    long wrong = 0;
    for (unsigned d : divisors) {
        const znn::FastDiv f = znn::make_fastdiv(d);
        auto check = [&](unsigned long n) { if (n + d < (1ul << 32) && znn::fdiv_any((unsigned)n, f) != n / d) ++wrong; };
        for (unsigned long q = 0; q * d < (1ul << 32); q = q < 4096 ? q + 1 : q + q / 64)
            for (long e = -4; e <= 4; ++e) if ((long)(q * d) + e >= 0) check(q * d + e);
        for (unsigned long n = 0; n < 300000; ++n) check(n);
        for (unsigned long n = 1; n < (1ul << 32); n += 104729) check(n);
    }
    printf("wrong %ld\n", wrong);
    return wrong != 0;
}
"""


def test_quotients_by_multiplication_are_exact(tmp_path):
    src, exe = tmp_path / "fastdiv.hip", tmp_path / "fastdiv"
    src.write_text(SOURCE)
    flags = [f for f in build.FLAGS if f != "-O3"]
    subprocess.run([build.HIPCC] + flags + ["-O1", "-w", "-o", str(exe), str(src)], check=True, cwd=os.path.dirname(build.CSRC))
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "wrong 0\n"
