"""The host rules that shape launches (csrc/fam_kernels.h, csrc/fam_ctx.h), evaluated on the
CPU: a small program that includes the headers, compiled for the host alone.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_26194_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

PROGRAM = r"""
#include <cstdio>
#include "fam_kernels.h"
#include "fam_ctx.h"
using namespace fam;

// the limiter's order is renewed wherever some items wait for others
static int order_of_items() {
  int bad = 0;
  for (int waves : {1, 2, 4}) {
    const int slots = SIMDS * waves;
    for (int items : {1, 1000, SIMDS - 1, SIMDS, SIMDS + 1, slots, slots + 1, 12000})
      for (int blocks : {1, 512, SIMDS, 2 * SIMDS, 4 * SIMDS, items}) {
        if (blocks > items) continue;
        const bool waits = blocks < items || items > slots;
        bad += starts_at_once(blocks, items, waves) == waits;
      }
  }
  return bad;
}

// a height is launched as set, but for the least where the model's is lower
static int set_heights() {
  int bad = 0;
  for (int model = 0; model < LEAST_H; ++model)
    for (int H = 1; H <= 64; ++H) {
      const int want = H <= LEAST_H && model > 0 ? std::min(H, model) : H;
      bad += launch_H(H, model) != want;
    }
  return bad;
}

// the sets of wave-speed maxima lie apart, and a launch's two in different lines
static int wave_speed_sets() {
  int bad = 0;
  for (bool spread : {true, false}) {
    const size_t len = spread ? ALPHA_SET : 2;
    for (int a = 0; a < 6; ++a) {
      const size_t x = alpha_set(spread, a), y = alpha_set(spread, (a + 1) % 6);
      bad += x + len > alpha_inst(spread) || x / ALPHA_STRIDE == y / ALPHA_STRIDE;
      for (int b = 0; b < a; ++b) {
        const size_t z = alpha_set(spread, b);
        bad += x < z + len && z < x + len;
      }
    }
  }
  return bad;
}

int main() {
  std::printf("order_of_items %d\nset_heights %d\nwave_speed_sets %d\n", order_of_items(), set_heights(),
              wave_speed_sets());
}
"""


@pytest.fixture(scope="module")
def violations(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return {name: int(count) for name, count in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("rule", ["order_of_items", "set_heights", "wave_speed_sets"])
def test_rule_holds(violations, rule):
    assert violations[rule] == 0
