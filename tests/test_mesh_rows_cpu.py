"""The row stride of the mesh passes' LDS planes (host rule, compiled with g++
against the library).

The kernels of half-width 4 take longer rows.  Wherever those leave room for too
few staged charges the plan keeps the general kernels' rows: M = 160, Kc = 40 in
either precision, M = 256, Kc = 32 in mixed and others were up to 1.9 times
slower with the longer ones.  What fits and how much memory the gather's
partials take is what the shorter rows give.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1303_4523_amd")

PROGRAM = r"""
#include "enuf_internal.h"
#include <cstdio>
#include <cstdlib>
using namespace enuf;
static int M, Kc, prec, ik;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (M %d Kc %d precision %d ik %d)\n", __LINE__, #x, M, Kc, \
                                              prec, ik); std::exit(1); } } while (0)
static MeshParams params(int p, int D) {
  MeshParams m{};
  m.M = M; m.Mp = M + 1; m.Mz = M + 1; m.Kc = Kc; m.nky = 2 * Kc - 1; m.win.p = p; m.cheb_deg = D; m.ik = ik;
  return m;
}
// the fewest chunks of the shorter rows, then the largest stage
static bool shorter(MeshParams &m, size_t lds) {
  for (int n = 1; n <= M / 2; ++n) {
    int rows = (M + n - 1) / n;
    rows += rows & 1;
    const int chunks = (M + rows - 1) / rows;
    if (n > 1 && rows < 8) return false;
    if (chunks > 1 && M - (chunks - 1) * rows < 8) continue;
    for (int stage = kStage; stage >= 32; stage /= 2) {
      m.rows = rows; m.nchunk = chunks; m.nslot = chunks > 1 ? 2 : 1; m.stage = stage;
      size_t f, x, b;
      mesh_lds_bytes(m, prec, &f, &x, &b);
      if (x > lds) return false;
      if (f <= lds && b <= lds) return true;
    }
  }
  return false;
}
int main() {
  const size_t budgets[] = {163840 - 256, 98304, 65536, 40000, 20000};
  for (size_t lds : budgets)
    for (M = 16; M <= 330; M += 2)
      for (int d = 4; d <= 8; ++d)
        for (prec = 0; prec < 2; ++prec)
          for (ik = 0; ik < 2; ++ik) {
            Kc = M / d;
            const int D = prec == 0 ? 14 : 9;
            MeshParams m = params(4, D), s = params(4, D);
            const bool fits = shorter(s, lds);
            CHECK(mesh_choose_rows(m, prec, lds) == fits);
            if (!fits) { CHECK(!mesh_win8(m) || m.rows == 0); continue; }
            size_t f, x, b;
            mesh_lds_bytes(m, prec, &f, &x, &b);
            CHECK(f <= lds && b <= lds && x <= lds);
            CHECK(m.nslot == s.nslot);
            if (mesh_win8(m)) {
              CHECK(m.stage >= (prec == 0 ? 64 : 128));
              CHECK(m.stage >= (prec == 0 ? 128 : 256) || m.stage >= s.stage);
            } else {
              CHECK(m.Mp == M + 1 && m.rows == s.rows && m.nchunk == s.nchunk && m.stage == s.stage);
            }
          }
  // with all of the LDS: the workloads' meshes take the longer rows, these do not
  struct { int M, Kc, prec, win8; } at[] = {{32, 8, 0, 1}, {64, 16, 0, 1}, {128, 32, 0, 1}, {128, 32, 1, 1},
      {160, 20, 0, 1}, {160, 40, 0, 0}, {160, 40, 1, 0}, {256, 32, 1, 0}, {128, 16, 1, 0}, {300, 37, 1, 0}};
  ik = 0;
  for (auto &a : at) {
    M = a.M; Kc = a.Kc; prec = a.prec;
    MeshParams m = params(4, prec == 0 ? 14 : 9);
    CHECK(mesh_choose_rows(m, prec, budgets[0]) && mesh_win8(m) == (a.win8 != 0));
  }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="no host toolchain")
def test_mesh_rows(tmp_path):
    src = tmp_path / "rows.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "rows"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PACKAGE, "csrc"), "-I", "/opt/rocm/include", str(src), "-L", PACKAGE, "-lenuf",
                    "-Wl,-rpath," + PACKAGE, "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined",
                    "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
