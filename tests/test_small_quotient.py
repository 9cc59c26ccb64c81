"""The float quotient of the simulation kernel (csrc/small_quotient.hip.inc) compiled for the host and compared with
integer division, for reciprocals one unit in the last place to either side of the exact one (what the hardware's may be)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cmath>
#include <cstdio>
#define __device__
#define __forceinline__ inline
static unsigned __umul24(unsigned a, unsigned b) { return (a & 0xffffffu) * (b & 0xffffffu); }
#include "small_quotient.hip.inc"

static unsigned long long wrong = 0;
static void check(unsigned x, unsigned d) {
  const float r = (float)(1.0 / d);
  const float near[3] = {r, std::nextafterf(r, 0.0f), std::nextafterf(r, 2.0f)};
  for (float rcp : near) {
    unsigned rest;
    const unsigned q = sim::divide_small(x, d, rcp, &rest);
    wrong += q != x / d || rest != x % d;
  }
}
int main() {
  for (unsigned d = 1; d <= 256; ++d) {
    const unsigned stride = d <= 4 || d == 255 || d == 256 ? 1u : 97u;
    for (unsigned x = 0; x < (1u << 22); x += stride) check(x, d); /* beyond the float range as well */
    for (unsigned k = 1; k <= (1u << 22) / d; k += stride) {       /* around multiples */
      check(k * d - 1u, d);
      check(k * d, d);
    }
    for (unsigned x = (1u << 21) - 600u; x < (1u << 21) + 600u; ++x) check(x, d);
    check(0xffffffffu, d);
  }
  std::printf("%llu\n", wrong);
}
"""


def test_small_quotient_is_exact(tmp_path):
    (tmp_path / "driver.cpp").write_text(DRIVER)
    exe = tmp_path / "driver"
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_2406_05221_amd", "csrc"),
                    "-o", str(exe), str(tmp_path / "driver.cpp")], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.strip() == "0"
