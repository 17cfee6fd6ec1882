"""The constants of the register-resident transforms (csrc/fft_reg.h): every twiddle
table entry against extended precision, to half an ulp of a double (rounded once)
plus the fixed-point series' own few units of 2^-61, for every length that a
factor or a lane pair's half can have.  A host program; no GPU.
"""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include "fft_reg.h"
using namespace qeh::regfft;
template <int N> void check() {
  const long double two_pi = 6.28318530717958647692528676655900577L;
  double worst = 0.0;
  for (int m = 0; m < N; ++m) {
    const long double ref[2] = {cosl(two_pi * m / N), -sinl(two_pi * m / N)};
    const double got[2] = {Tw<N>::t.re[m], Tw<N>::t.im[m]};
    for (int i = 0; i < 2; ++i) {
      const double a = std::fabs((double)ref[i]);
      if (a < 1e-15) {   // an exact zero
        if (got[i] != 0.0) worst = 1e9;
        continue;
      }
      const double ulp = std::nextafter(a, 2.0) - a;
      worst = std::fmax(worst, (double)(fabsl(got[i] - ref[i]) / ulp));
    }
  }
  std::printf("%d %.3f\n", N, worst);
}
template <int... N> void all() { (check<N>(), ...); }
int main() {
  all<1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 50,
      54, 60, 64, 72, 80, 90>();
}
"""


def test_twiddles_to_half_an_ulp(tmp_path):
    src = tmp_path / "tables.hip"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "tables")
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    csrc = os.path.join(ROOT, "paper_2104_10502_amd", "csrc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I" + csrc, "-o", exe,
                    str(src)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 31
    for n, worst in rows:
        # rounded once; ten units of 2^-61 against an ulp of at least 2^-56 (sin(2 pi / 90) > 2^-4)
        assert float(worst) <= 0.5 + 10 * 2.0 ** -5, (n, worst)
