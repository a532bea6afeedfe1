"""The quantisation kernels' short quotient (csrc/e4m3.hpp) against the division, exhaustively, on the host: the two functions the
kernels use are compiled for the CPU and run over every case that the comment beside them claims."""
import os
import subprocess

from paper_2512_07710_amd.build import HIPCC

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "e4m3.hpp"
#include <cmath>
#include <cstdio>
#include <cstring>
static float from_bits(uint32_t b) { float f; memcpy(&f, &b, 4); return f; }
static uint32_t to_bits(float f) { uint32_t b; memcpy(&b, &f, 4); return b; }
int main() {
    long cases = 0, wrong = 0;
    for (int which = 0; which < 3; ++which)                    // scales at the middle and just inside both ends of the range
        for (uint32_t ma = 0; ma < 128; ++ma) {                // bf16 significand of the group's largest value
            float amax = from_bits((127u << 23) | (ma << 16));
            float s = amax / 448.0f;
            if (which == 1) while (s * 0.5f > moe355::SCALE_MID_MIN) { s *= 0.5f; amax *= 0.5f; }
            if (which == 2) while (s * 2.0f < moe355::SCALE_MID_MAX) { s *= 2.0f; amax *= 2.0f; }
            for (int off = -2; off <= 2; ++off) {              // the hardware's estimate: up to 2 ulp off
                const float inv = moe355::refined_reciprocal(s, from_bits(to_bits(1.0f / s) + off));
                for (uint32_t mv = 0; mv < 128; ++mv)
                    for (int e = 0; e < 20; ++e)               // quotients from 448 down to below the smallest non-zero code's half
                        for (int sign = 0; sign < 2; ++sign) {
                            float v = from_bits((to_bits(amax) & 0x7F800000u) | (mv << 16));
                            v = ldexpf(v, -e);
                            if (v > amax) continue;
                            if (sign) v = -v;
                            const float q = moe355::corrected_quotient(v, s, inv);
                            ++cases;
                            wrong += to_bits(q) != to_bits(v / s);
                        }
                for (int sign = 0; sign < 2; ++sign) {
                    const float z = sign ? -0.0f : 0.0f;
                    wrong += to_bits(moe355::corrected_quotient(z, s, inv)) != to_bits(z);
                }
            }
        }
    printf("%ld %ld\n", cases, wrong);
    return 0;
}
"""


def test_short_quotient_equals_the_division(tmp_path):
    src, exe = tmp_path / "quotient.hip", tmp_path / "quotient"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_2512_07710_amd", "csrc"), str(src), "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert int(out[0]) > 9_000_000 and int(out[1]) == 0, out
