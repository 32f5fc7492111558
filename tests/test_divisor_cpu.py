"""The multiplication that replaces the kernels' integer divisions (struct
Divisor in fa_common.h), compiled for the host and compared with division."""
import os
import subprocess

from paper_2608_18656_amd import build as hip_build

MAIN = r"""
#include "fa_common.h"
#include <cstdio>
int main() {
    unsigned long long bad = 0, x = 88172645463325252ull;
    auto check = [&](unsigned n, unsigned d) {
        const fa::Divisor v(d);
        bad += (unsigned)(((unsigned long long)n * v.m) >> v.shift) != n / d;
    };
    for (unsigned d = 1; d < 3000; ++d)
        for (unsigned k = 0; k < 40; ++k) {
            check(k, d);
            check(k * d, d);
            check(k * d + d - 1, d);
            check(0x7fffffffu - k, d);
        }
    for (int i = 0; i < 2000000; ++i) {
        x ^= x << 13; x ^= x >> 7; x ^= x << 17;
        const unsigned d = (unsigned)(x & 0x7fffffffu) >> (x >> 59);
        check((unsigned)(x >> 32) & 0x7fffffffu, d ? d : 1u);
    }
    std::printf("%llu\n", bad);
}
"""


def test_divisor(tmp_path):
    src, exe = tmp_path / "d.hip", tmp_path / "d"
    src.write_text(MAIN)
    subprocess.run([hip_build.hipcc(), *hip_build.HIPCC_FLAGS, "-w", "-I", hip_build.CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="")
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, env=env).stdout.strip() == "0"
