"""The writer's quotients from one reciprocal (CPU).

The quantizer divides every bf16 value of a group by the group's fp32 scale s,
correctly rounded.  The kernel computes r = RN(1 / s) once and each quotient as
q = RN(x r) corrected by the exact remainder, RN(q + RN(x - q s) r) with fused
multiply-adds.  This compares that with the IEEE division for every pair of
mantissas (powers of two scale through): 128 bf16 mantissas x 2^23 scales.
"""
import os
import subprocess

import pytest

SRC = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>
int main() {
    long differ[4] = {0, 0, 0, 0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 4; ++t)
        threads.emplace_back([&differ, t] {
            for (uint32_t m = t; m < (1u << 23); m += 4) {
                const uint32_t bits = 0x3F800000u | m;
                float s;
                std::memcpy(&s, &bits, 4);
                const float r = 1.0f / s;
                for (int j = 128; j < 256; ++j) {
                    const float x = j / 128.0f, q = x * r;
                    differ[t] += std::fmaf(std::fmaf(-q, s, x), r, q) != x / s;
                }
            }
        });
    for (auto& t : threads) t.join();
    std::printf("%ld\n", differ[0] + differ[1] + differ[2] + differ[3]);
}
"""


def test_corrected_quotient_is_the_division(tmp_path):
    with open("/proc/cpuinfo") as f:
        if " fma " not in f.read():
            pytest.skip("no fused multiply-add on this CPU")
    src, exe = tmp_path / "q.cpp", tmp_path / "q"
    src.write_text(SRC)
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-pthread", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300, cwd=os.fspath(tmp_path))
    assert int(out.stdout) == 0
