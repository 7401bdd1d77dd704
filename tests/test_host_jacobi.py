"""CPU test of the subspace eigensolver's rotation: with root and reciprocal estimates that are off
by up to 2^-23, as the hardware's may be, the angle is as good as one from exact roots and divisions,
for pairs of every grading and over the whole range of magnitudes."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <cstdint>
#include "jacobi.hpp"
static uint64_t g_s = 1;
static uint64_t next() {  // splitmix64
  uint64_t z = (g_s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
static double uniform() { return (double)(next() >> 11) * 0x1p-53 * 2.0 - 1.0; }
struct Est {  // the true value, off by up to 2^-23
  static double off(long double v) { return (double)(v * (1.0L + 0x1p-23L * uniform())); }
  static double rsq(double x) { return off(1.0L / std::sqrt((long double)x)); }
  static double rcp(double x) { return off(1.0L / (long double)x); }
};
int main() {
  double et = 0, ec = 0, eo = 0;
  for (int i = 0; i < 400000; ++i) {
    const int e = (int)(next() % 1960) - 940;  // magnitude of the pair: 2^-940 .. 2^1019
    double app = std::ldexp(uniform(), e), aqq = std::ldexp(uniform(), e), apq = std::ldexp(uniform(), e);
    switch (i % 4) {
      case 1: apq = std::ldexp(apq, -(int)(next() % 50)); break;                      // weak coupling
      case 2: aqq = app + std::ldexp(apq, (int)(next() % 60) - 30 - 4); break;        // close together
      case 3: app = std::ldexp(app, -(int)(next() % 50)); apq = std::ldexp(apq, -(int)(next() % 40)); break;  // graded
    }
    if (!(std::fabs(apq) > 1e-300) || !std::isfinite(aqq)) continue;
    double c, s;
    dmrg::jacobi_rotation<Est>(app, aqq, apq, c, s);
    // the difference as the solver rounds it, everything after it in long double
    const long double x = (long double)(aqq - app), y = 2.0L * apq, r = std::hypot(x, y);
    const long double t = (x >= 0 ? y : -y) / (std::fabs(x) + r), cw = 1.0L / std::sqrt(1.0L + t * t), sw = t * cw;
    if (!(std::isfinite(c) && std::isfinite(s))) { std::printf("not finite at %d\n", i); return 1; }
    if (std::fabs(sw) > 1e-290L) et = std::fmax(et, (double)std::fabs((s - sw) / sw));
    ec = std::fmax(ec, (double)std::fabs((c - cw) / cw));
    eo = std::fmax(eo, (double)std::fabs((long double)c * c + (long double)s * s - 1.0L));
  }
  std::printf("%.17g %.17g %.17g\n", et, ec, eo);
}
"""


def test_rotation_has_full_precision(tmp_path):
    src, exe = tmp_path / "rot.cpp", tmp_path / "rot"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2609_09990_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    es, ec, eo = (float(x) for x in r.stdout.split())
    print(es, ec, eo)
    u = 2.0 ** -53
    # s: h, r, den, inv, y inv, t c one rounding each and w's half: 6.5 u, and the second-order
    # remainders of the Newton steps (2^-46)^2; an angle of one step is off by 2^-46 = 128 u
    assert es <= 8 * u
    assert ec <= 3 * u  # w (half), the last step's product and sum
    assert eo <= 8 * u
