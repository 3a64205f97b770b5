"""The one-wave cell kernel's plane accesses stay inside the wave's LDS slab:
lanes without a plane of their own read too (their values are not used), so
every lane's address must be in range at every degree and precision.  Checked
at compile time from the expression that the kernel addresses with."""

import os
import subprocess

import pytest

PLANES = """
#include "cell_valu.h"
using namespace pawfe;
template <typename T, int NP, int NQ>
constexpr bool in_slab() {
  using W = Wave<T, NP, NQ>;
  for (int lane = 0; lane < 64; ++lane) {
    if (W::plane_at(lane) < 0 || W::plane_at(lane) + (NQ * NQ - 1) * NP * W::CB >= W::slab) return false;
    // the last line of every existing plane is the last of its own elements
    const int s = (lane / W::CB) % W::PS;
    if (s < NP && W::plane_at(lane) != s * W::CB + lane % W::CB) return false;
  }
  return true;
}
static_assert(in_slab<T_, NP_, NP_ + 1>(), "plane access outside the slab");
"""


@pytest.mark.parametrize("p", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("t", ["float", "double"])
def test_plane_accesses_stay_in_the_slab(tmp_path, p, t):
    from paper_2604_26037_amd import build
    src = tmp_path / "planes.hip"
    src.write_text(PLANES.replace("T_", t).replace("NP_", str(p + 1)))
    cmd = [build.hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-fsyntax-only",
           "-I", build.INCLUDE, "-I", build.CSRC, str(src)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=120, cwd=os.path.dirname(build.CSRC))
    assert r.returncode == 0, r.stderr[-2000:]
