"""CPU test of the voice-hits screen's error bound (csrc/wnw_screen.h): over all scales of queries and keys
that the range check accepts, a matrix unit that flushes every subnormal input, product and sum, and
truncates every sum, stays inside the bound."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MODEL = r"""
#include "wnw_screen.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

using namespace wnw;

static float bf16(double v)
{
    float f = (float)v;
    unsigned u;
    std::memcpy(&u, &f, 4);
    u &= 0xffff0000u;
    std::memcpy(&f, &u, 4);
    return f;
}
// towards zero to fp32, subnormals flushed
static float unit(double v)
{
    float f = (float)v;
    if (std::fabs((double)f) > std::fabs(v)) f = std::nextafterf(f, 0.f);
    return std::fabs(f) < 0x1p-126f ? 0.f : f;
}

int main()
{
    std::mt19937 rng(1);
    std::normal_distribution<double> normal;
    long tested = 0;
    double worst = 0.0;
    for (int iq = -130; iq <= 70; iq += 2)
        for (int ik = -130; ik <= 70; ik += 2)
            for (int rep = 0; rep < 3; ++rep) {
                float q[128], k[128], S = 0.f, q1 = 0.f, kmax = 0.f;
                for (int d = 0; d < 128; ++d) {
                    // rep 1: magnitudes over many octaves; rep 2: a few large key elements
                    const double wide = rep == 1 ? std::exp2(-20.0 * std::fabs(normal(rng))) : 1.0;
                    const double big = rep == 2 && d % 40 == 7 ? 500.0 : 1.0;
                    q[d] = bf16(std::ldexp(normal(rng) * wide, iq));
                    k[d] = bf16(std::ldexp(normal(rng) * big, ik));
                    // S from a larger key of the same channel now and then
                    S += std::fabs(q[d]) * std::fabs(k[d]) * (d % 3 ? 1.f : 4.f);
                    q1 += std::fabs(q[d]);
                    kmax = std::fmax(kmax, std::fabs(k[d]));
                }
                if (!screen_in_range(S, q1, kmax)) continue;
                ++tested;
                long double exact = 0;
                float a = 0.f;
                for (int d = 0; d < 128; ++d) {
                    exact += (long double)q[d] * k[d];
                    a = unit((double)a + unit((double)unit(q[d]) * unit(k[d])));
                }
                const double m = (double)VF_GAMMA * S, err = (double)std::fabs((long double)a - exact);
                worst = std::fmax(worst, err / m);
                if (!(err <= m)) {
                    std::printf("2^%d 2^%d %d: error %g over the bound %g\n", iq, ik, rep, err, m);
                    return 1;
                }
            }
    const float inf = INFINITY, nan = NAN;
    for (float v : {inf, nan, 0.f})
        if (screen_in_range(v, 1.f, 1.f)) return std::printf("accepts %g\n", v), 1;
    for (float v : {inf, nan})
        if (screen_in_range(1.f, v, 1.f) || screen_in_range(1.f, 1.f, v)) return std::printf("accepts %g\n", v), 1;
    std::printf("ok %ld tested, worst %g of the bound\n", tested, worst);
    return tested < 10000;
}
"""


def test_screen_bound(tmp_path):
    src, exe = tmp_path / "bound.cpp", tmp_path / "bound"
    src.write_text(MODEL)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2608_22704_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
