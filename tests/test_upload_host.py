"""An upload for which the host has no memory left to put its tables together
takes them one by one: nothing is thrown through the C call (host only; without
a device the copies then fail with an error code)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_11709_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <new>
#include "%(root)s/include/xrd.h"
#include "xrd_internal.h"
namespace xrd {
void launch_fill_i32(int32_t *, int64_t, int32_t, hipStream_t) {}
}  // namespace xrd
static bool armed = false;
static bool refuse(size_t n) {  // the first allocation of a table's size
  const bool no = armed && n >= 1024;
  if (no) armed = false;
  return no;
}
void *operator new(size_t n) {
  void *p = refuse(n) ? nullptr : std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void *operator new[](size_t n) { return operator new(n); }
void *operator new(size_t n, const std::nothrow_t &) noexcept { return refuse(n) ? nullptr : std::malloc(n ? n : 1); }
void *operator new[](size_t n, const std::nothrow_t &t) noexcept { return operator new(n, t); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }
int main() {
  const double lat[6] = {4, 4, 4, 90, 90, 90}, lo = 10, hi = 60;
  const int64_t off[2] = {0, 1};
  static double any[64];
  xrd_batch_desc d{};
  d.n_crystals = 1;
  d.n_species = 1;
  d.lattice = lat;
  d.atom_offset = off;
  d.two_theta_min = &lo;
  d.two_theta_max = &hi;
  d.wavelength = 1.54184;
  d.merge_tol = 1e-5;
  d.frac = d.occ = d.bfac = d.sf_coeff = any;
  d.species = (const int32_t *)any;
  xrd_batch *b = nullptr;
  if (xrd_batch_create(&d, &b) != XRD_OK) return 1;
  xrd_sizes z;
  if (xrd_batch_sizes(b, &z) != XRD_OK) return 1;
  void *ws = std::aligned_alloc(256, (size_t)(z.workspace_bytes + 255) / 256 * 256);
  armed = true;
  try {
    const int rc = xrd_batch_upload(b, ws);
    std::printf("%%s %%s\n", rc == XRD_OK || rc == XRD_ERR_HIP ? "returned" : "refused", armed ? "untried" : "tried");
  } catch (const std::bad_alloc &) {
    std::printf("thrown\n");
  }
  xrd_batch_destroy(b);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/lib/libamdhip64.so"),
                    reason="g++ or the HIP runtime library not available")
def test_no_memory_to_put_tables_together(tmp_path):
    (tmp_path / "m.cpp").write_text(PROGRAM % {"root": ROOT})
    exe = str(tmp_path / "m")
    # the stand-in above comes before the ones that abort
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", "-I", CSRC,
                           str(tmp_path / "m.cpp"), os.path.join(CSRC, "api.cpp"),
                           os.path.join(ROOT, "tests", "sanitize", "launch_stubs.cpp"), "-L/opt/rocm/lib",
                           "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-multiple-definition", "-lpthread",
                           "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60, env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    assert out.returncode == 0 and out.stdout.split() == ["returned", "tried"], out
