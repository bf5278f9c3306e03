"""The position codes of angle keys: never decreasing with the key, and inside
their bits, for epipoles everywhere (a small program around the header, on the
CPU).  Windows of keys are searched as windows of codes, so a code that went
back would lose candidates."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_18401_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "epm_internal.h"
using namespace epm;

int main() {
  srand(1);
  long bad = 0, arcs = 0;
  for (int t = 0; t < 300; ++t) {
    PairDev pd{};
    pd.kappa = t % 50 == 7 ? -1.0 : 1.0;  // without a pencil: the whole circle
    pd.s = 1e-3;
    pd.cx = 300 + rand() % 4000;
    pd.cy = 300 + rand() % 4000;
    // the epipole in normalised coordinates: the centre, inside, beside, far, infinite
    const double a = rand() % 1000 * 0.00628;
    const double r = t % 5 == 0 ? 0.0 : t % 5 == 1 ? 1e4 : (rand() % 1000) / 100.0;
    const double e[3] = {r * cos(a) + (t % 7 == 0), r * sin(a), t % 7 == 0 ? 0.0 : 1.0};
    const double n = sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]);
    for (int k = 0; k < 3; ++k) pd.e[k] = e[k] / n;
    // u, v: an orthonormal basis of the lines through it
    const int h = fabs(pd.e[0]) < 0.5 ? 0 : 1;
    double q = 0.0;
    for (int k = 0; k < 3; ++k) {
      pd.u[k] = (k == h) - pd.e[h] * pd.e[k];
      q += pd.u[k] * pd.u[k];
    }
    for (int k = 0; k < 3; ++k) pd.u[k] /= sqrt(q);
    for (int k = 0; k < 3; ++k)
      pd.v[k] = pd.e[(k + 1) % 3] * pd.u[(k + 2) % 3] - pd.e[(k + 2) % 3] * pd.u[(k + 1) % 3];
    set_key_arc(pd);
    arcs += pd.arc.arc_len != 0u;
    const uint32_t off = pd.arc.arc_len ? arc_side(pd.arc.arc_len) : 1u << 20;
    const uint32_t near = pd.arc.arc_len ? arc_near(pd.arc.arc_len) : 1u;
    const uint32_t end = 1u << kCentreBits;
    uint32_t last = 0;
    for (uint64_t k = 0; k < 0x100000000ull; k += 1 + rand() % 300000) {
      const uint32_t c = position_code(pd.arc, (uint32_t)k);
      bad += c < last || c >= end;
      last = c;
    }
    const uint32_t top = off + pd.arc.arc_len;
    const uint32_t edge[] = {1u, off - near - 1, off - near, off - near + 1, off, off + 1, top - 1,
                             top, top + 1, top + near - 1, top + near, top + near + 1,
                             0xFFFFFFFEu, 0xFFFFFFFFu};
    for (uint32_t k : edge)
      if (k > 0)
        bad += position_code(pd.arc, k) < position_code(pd.arc, k - 1) || position_code(pd.arc, k) >= end;
  }
  printf("%ld wrong, %ld arcs\n", bad, arcs);
  return bad != 0 || arcs < 50;
}
"""


def test_codes_never_decrease(tmp_path):
    src, exe = tmp_path / "codes.cpp", tmp_path / "codes"
    src.write_text(PROGRAM)
    r = subprocess.run(["hipcc", "-x", "hip", "-O1", "-std=c++17", "--offload-arch=gfx950",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    if r.returncode != 0 and "No such file" in r.stderr and "hipcc" in r.stderr:
        pytest.skip("no hipcc")
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
