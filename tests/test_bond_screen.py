"""The FP32 screen of the structure analyses (csrc/bond_screen.h), compiled for
the CPU: every pair inside the cutoff is noted, inside the box and across its
faces, edges and corners, for edges about powers of two (where a copy is worst)
and from three cells to 4096 along an axis; the error never passes the derived
bound, half of the margin."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <initializer_list>
#include <stdint.h>
#include <stdio.h>
#define __device__
#define __forceinline__ inline
#include "bond_screen.h"
static uint64_t state = 88172645463325252ull;
static double uniform() {  // xorshift64, 53 bits
  state ^= state << 13;
  state ^= state >> 7;
  state ^= state << 17;
  return (double)(state >> 11) / 9007199254740992.0;
}
int main() {
  int bad = 0;
  const double edges[] = {3.0001, 7.9999, 8.0001, 15.999, 16.001, 63.99, 64.01, 100.0, 511.9, 512.1, 4095.9, 4097.0};
  for (double edge : edges)
    for (int mixed = 0; mixed < 2; ++mixed)
      for (double rc : {0.9999, 1e-3 * edge}) {
        const double box[3] = {edge, mixed ? 3.3 * rc : edge, mixed ? 0.5 * edge > 3 * rc ? 0.5 * edge : edge : edge};
        double side[3];
        for (int k = 0; k < 3; ++k) {
          double q = floor(box[k] / (rc * (1.0 + 1e-10)));
          side[k] = box[k] / (q > 4096.0 ? 4096.0 : q);
        }
        const float r2 = mdpl::screen_r2(box, side, rc * rc);
        double worst = 0.0;
        for (int t = 0; t < 40000; ++t) {
          // j near the faces half of the time, i at almost the cutoff from it
          double xj[3], d[3], s = 0.0;
          for (int k = 0; k < 3; ++k) {
            xj[k] = uniform() * box[k];
            if (t & 1 << k) xj[k] = t & 8 ? uniform() * rc : box[k] - uniform() * rc;
            if (!(xj[k] < box[k])) xj[k] = 0.0;
            d[k] = t % 5 == 0 && k ? 0.0 : uniform() - 0.5;
            s += d[k] * d[k];
          }
          const double len = rc * (1.0 - 1e-12 - 1e-6 * (t % 3) * uniform());
          float c[3];
          for (int k = 0; k < 3; ++k) {
            double xi = xj[k] + d[k] * len / sqrt(s);
            // the folded particle, and the side of the box on which it finds j
            const int w = xi < 0.0 ? 1 : (xi >= box[k] ? -1 : 0);
            xi += w > 0 ? box[k] : (w < 0 ? -box[k] : 0.0);
            if (!(xi >= 0.0 && xi < box[k])) xi = 0.0;
            c[k] = mdpl::screen_image((float)xi, box[k], w) - (float)xj[k];
          }
          const float d2 = mdpl::screen_d2(c[0], c[1], c[2]);
          if (!(d2 <= r2)) ++bad;
          const double e = ((double)d2 - len * len) / ((double)r2 - rc * rc);
          worst = e > worst ? e : worst;
        }
        printf("edge %g rc %g box %g %g: margin used %.3f\n", edge, rc, box[1], box[2], worst);
        if (worst > 0.5) ++bad;
      }
  printf("%d wrong\n", bad);
  return bad != 0;
}
"""


def test_screen_notes_every_bond(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "screen.cpp", tmp_path / "screen"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_1704_03329_amd", "csrc")
    subprocess.run([gxx, "-std=c++17", "-O1", "-ffp-contract=off", "-I", csrc, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout[-4000:])
    assert r.returncode == 0, r.stdout[-4000:]
