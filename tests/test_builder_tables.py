"""Host tables of the operator builder where an atom has no support row (its
radius holds no Gauss point): every device read at the atom's first work item
has to stay inside the table, also for the last atom.  A small host program
runs the builder and checks the ranges; the kernels run the same operator in
test_gpu_empty_support.py."""

import os
import subprocess

import pytest

MAIN = r"""
#include <cstdio>
#include <vector>
#include "internal.h"
int main() {
  pawfe_op_desc d{};
  for (int k = 0; k < 3; ++k) { d.ncell[k] = 3; d.box[k] = 4.8; }
  d.degree = 3;
  d.nq1d = 5;
  std::vector<double> v(27 * 125, -0.5);
  d.veff_q = v.data();
  const int na = 3;
  const double pos[9] = {0.4, 0.5, 0.6, 2.0, 2.2, 3.1, 3.9, 1.1, 0.7};
  int empty = 0;
  for (int mask = 1; mask < 8; ++mask) {
    double rcut[3];
    for (int a = 0; a < na; ++a) rcut[a] = (mask >> a) & 1 ? 1.1 : 1e-6;
    const int32_t np[3] = {1, 2, 1}, l[4] = {0, 0, 0, 0}, m[4] = {0, 0, 0, 0};
    const double sig[4] = {0.4, 0.4, 0.3, 0.5}, D[6] = {1, 1, 0, 0, 1, 1};
    d.natoms = na; d.pos = pos; d.rcut = rcut; d.nproj = np; d.proj_l = l; d.proj_m = m; d.proj_sigma = sig;
    d.dH = D; d.dS = D;
    pawfe_op op;
    if (pawfe::build_host(&d, &op) != PAWFE_OK) { std::printf("build failed\n"); return 1; }
    for (int a = 0; a < na; ++a) {
      const int i0 = op.item_ptr[a], ni = op.item_ptr[a + 1] - i0;
      empty += ni == 0;
      if ((ni == 0) != !((mask >> a) & 1)) { std::printf("support of atom %d\n", a); return 1; }
      if (i0 >= (int)op.item_poff.size()) { std::printf("mask %d atom %d: offset %d of %zu\n", mask, a, i0, op.item_poff.size()); return 1; }
      if (op.gq_ptr[a] > op.gq_ptr[a + 1] || op.gq_ptr[a + 1] > (int)op.gq_row.size()) return 1;
    }
  }
  return empty == 9 ? 0 : 1;
}
"""


def test_offsets_of_atoms_without_support(tmp_path):
    from paper_2604_26037_amd import build
    if not os.path.exists(build.LIB):
        pytest.skip("libpawfe.so not built")
    src, exe = tmp_path / "tables.hip", tmp_path / "tables"
    src.write_text(MAIN)
    cmd = [build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "-I", build.INCLUDE, "-I", build.CSRC, str(src),
           "-o", str(exe), "-L" + build.PKG, "-l:" + os.path.basename(build.LIB), "-Wl,-rpath," + build.PKG]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
