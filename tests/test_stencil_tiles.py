"""The stencil's launch shapes against the LDS that they ask for: no lane's read
or write lies outside its plane buffer.  The shapes come from the library's own
rule (host code), compiled here by itself; the kernel's index ranges are written
out below."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")

# A lane's neighbours reach 6 rows and columns; the band starts at row 6 and
# column 6 of its plane buffer.  Paired rows start at rows 0, 2, 4, ... of the
# band and read rows -6 .. 7 about their first; paired columns start at columns
# 0, 2, ... and read columns -6 .. 7.
SWEEP = r"""
#include <cstdio>
#include "stencil_impl.h"
using namespace xls;
using namespace xls::stencil_detail;
void xls::fail(int code, const std::string& msg) { throw Error{code, msg}; }
int main() {
  long n = 0, bad = 0, odd = 0;
  const int ext[] = {1, 2, 3, 7, 12, 16, 21, 24, 32, 33, 40, 47, 61, 64, 67, 68, 69, 80, 96, 100, 101, 115, 116};
  const int nys[] = {1, 9, 21, 23, 64, 110}, tys[] = {0, 1, 3, 5, 7, 8, 11, 15, 16};
  const long cols[] = {1, 229, 5000};
  for (int nx : ext) for (int ny : nys) for (int nz : {1, 14, 57}) for (int elem : {4, 8}) for (int nproj : {0, 4, 1600})
  for (long c : cols) for (int per : {0, 1}) for (int tz : {-1, 0}) for (int block : {0, 256, 512}) for (int ty : tys)
  for (int nv : {0, 1, 2}) {
    StencilLaunch cfg;
    cfg.block = block; cfg.ty = ty; cfg.tz = tz; cfg.nv = nv;
    const TileChoice t = choose_tiles(nx, ny, nz, elem, nproj, c, per, cfg);
    try { check_tiles(t, nx, per, elem); } catch (const Error&) { continue; }
    const long plane = (static_cast<long>(t.smem) / elem / t.nv - nproj) / 2;
    long last = 0;
    for (int tyv : {t.ty, ny - (t.nyt - 1) * t.ty}) {
      const int row = t.pk == kRowPairs ? (tyv - 1) / 2 * 2 + 1 : tyv - 1;  // a pair reads for both of its rows
      const int col = t.pk >= kXPairs ? (nx - 1) / 2 * 2 + 1 : nx - 1;
      last = std::max<long>(last, static_cast<long>(row + 2 * R) * t.ws + R + nx - 1);         // y neighbours
      last = std::max<long>(last, static_cast<long>(tyv - 1 + R) * t.ws + col + 2 * R);        // x neighbours
      if (col + 2 * R >= t.ws) last = plane;
    }
    ++n;
    odd += t.pk == kRowPairs && t.ty % 2;
    if (last >= plane && bad++ < 5)
      std::printf("nx %d ny %d nz %d elem %d nproj %d cols %ld periodic %d: block %d ty %d nv %d pk %d reads cell %ld of %ld\n",
                  nx, ny, nz, elem, nproj, c, per, t.block, t.ty, t.nv, t.pk, last, plane);
  }
  std::printf("shapes %ld odd paired bands %ld outside %ld\n", n, odd, bad);
  return bad != 0 || n == 0 || odd == 0;
}
"""


# Vectors per tile of FP32 launches on both sides of each condition of the rule:
# rows of whole sectors or past 64 points, enough workgroups, and LDS for two
# workgroups per CU; two-vector tiles halve the z range until a launch has six
# thousand of them
RULE = r"""
#include <cstdio>
#include "stencil_impl.h"
using namespace xls;
using namespace xls::stencil_detail;
void xls::fail(int code, const std::string& msg) { throw Error{code, msg}; }
int main() {
  const int shapes[][7] = {  // nx, ny, nz, columns, coefficients, vectors, z chunks of two-vector tiles
      {64, 64, 64, 480, 1600, 2, 2}, {64, 64, 64, 300, 1600, 1, 0}, {53, 61, 47, 900, 800, 1, 0}, {60, 62, 62, 694, 800, 1, 0},
      {65, 67, 62, 445, 1000, 2, 2}, {65, 67, 62, 200, 1000, 1, 0}, {69, 68, 69, 443, 1000, 2, 2}, {69, 68, 69, 200, 1000, 1, 0},
      {77, 78, 75, 700, 1600, 2, 2}, {77, 78, 75, 1000, 1600, 2, 1}, {85, 85, 85, 400, 1600, 2, 2}, {85, 85, 85, 500, 9000, 1, 0},
      {64, 64, 64, 1500, 1600, 2, 2}, {64, 64, 64, 1600, 1600, 2, 1}, {48, 48, 48, 1200, 1600, 2, 1}};
  int bad = 0;
  for (const auto& s : shapes) {
    const TileChoice t = choose_tiles(s[0], s[1], s[2], 4, s[4], s[3], 0, StencilLaunch{});
    if (t.nv != s[5] || (s[6] && t.nzt != s[6])) ++bad, std::printf("%d %d %d x %d: %d vectors, %d chunks\n", s[0], s[1], s[2], s[3], t.nv, t.nzt);
  }
  return bad != 0;
}
"""


def run_program(tmp_path, source):
    src, exe = tmp_path / "prog.hip", tmp_path / "prog"
    src.write_text(source)
    csrc = os.path.join(ROOT, "paper_2609_13115_amd", "csrc")
    hipcc = HIPCC if os.path.exists(HIPCC) else shutil.which("hipcc")
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-Wno-unused-result", "-I", csrc,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, timeout=240)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout


needs_hipcc = pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="no hipcc")


@needs_hipcc
def test_tiles_stay_inside_their_plane_buffers(tmp_path):
    run_program(tmp_path, SWEEP)


@needs_hipcc
def test_vectors_per_tile_of_fp32_launches(tmp_path):
    run_program(tmp_path, RULE)
