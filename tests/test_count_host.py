"""Index arithmetic of the sweeps at the largest sizes (no GPU): a program compiled
against the library's headers runs the host side of the functions that the kernels
share."""
import os
import subprocess

import pytest

from paper_2010_10272_amd import build

PROGRAM = r"""
#include <stdio.h>
#include "hg_count.h"
#include "hg_lp.h"
using namespace hg;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  const int most = 0x7fffffff;
  // units that cover counts just below 2^31
  for (int per : {32, 128, 256, 4096}) {
    CHECK(units_of(most, per) == (int)(2147483648LL / per));
    CHECK(units_of(most - per, per) == (int)(2147483648LL / per) - 1);
    CHECK(units_of(1, per) == 1 && units_of(per, per) == 1 && units_of(per + 1, per) == 2);
  }
  // a run of any length below 2^31 is walked to its end, every place in one step
  for (int total : {1, 255, 256, 257, 65536, most - 256, most - 255, most - 1, most}) {
    long long steps = 0, hits = 0, places = 0;
    for (RunPlace s = 0; run_left(s, total); s += kCountStep) {
      CHECK(++steps <= 2147483648LL / kCountStep);
      hits += in_step(total - 1, s) < kCountStep;
      places += run_left(s + kCountStep - 1, total) ? kCountStep : (long long)total - s;
    }
    CHECK(steps == ((long long)total + kCountStep - 1) / kCountStep);
    CHECK(hits == 1 && places == total);
  }
  printf("ok\n");
  return 0;
}
"""


def run_host(tmp_path, program):
    src = tmp_path / "host.hip"
    src.write_text(program)
    exe = str(tmp_path / "host")
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-fwrapv", "-std=c++17", "-w",
                    "-I" + build.CSRC, str(src), "-o", exe], check=True, timeout=300)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_sizes_near_two_to_the_31(tmp_path):
    r = run_host(tmp_path, PROGRAM)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
