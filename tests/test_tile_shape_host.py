"""The tile shape that the structure factors are launched with (host only, the
device launches replaced by stand-ins): the caller's as it is, the default one
open to the launch's own choice."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_11709_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "%(root)s/include/xrd.h"
#include "xrd_internal.h"
namespace xrd {
void launch_sf(bool, bool, const SfItem *, int64_t, int64_t, const CrystalPlan *, const int64_t *, const int16_t *,
               const int16_t *, const int16_t *, const double *, const double *, const AtomRec *, const SpeciesRun *,
               const int32_t *, const double *, const CoeffF *, void *, void *, double *, void *, int rpt, hipStream_t) {
  std::printf(" %%d%%s", rpt & ~kTileFixed, rpt & kTileFixed ? "!" : "");
}
}  // namespace xrd
int main() {
  const double lat[6] = {4, 4, 4, 90, 90, 90}, lo = 10, hi = 60;
  const int64_t off[2] = {0, 1};
  static double any[64];
  for (int rpt : {0, 1, 2, 4}) {
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
    d.sf_rpt = rpt;
    xrd_batch *b = nullptr;
    if (xrd_batch_create(&d, &b) != XRD_OK) return 1;
    alignas(256) static char ws[256];
    xrd_refl r{};
    r.refl_offset = (int64_t *)any;
    r.h = r.k = r.l = (int16_t *)any;
    r.q = r.two_theta = r.lp = any;
    xrd_structure_factors(b, ws, &r, any, any, any);
    xrd_batch_destroy(b);
  }
  std::printf("\n");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/lib/libamdhip64.so"),
                    reason="g++ or the HIP runtime library not available")
def test_given_shape_is_launched(tmp_path):
    (tmp_path / "m.cpp").write_text(PROGRAM % {"root": ROOT})
    exe = str(tmp_path / "m")
    # the stand-in above comes before the ones that abort
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", "-I", CSRC,
                           str(tmp_path / "m.cpp"), os.path.join(CSRC, "api.cpp"),
                           os.path.join(ROOT, "tests", "sanitize", "launch_stubs.cpp"), "-L/opt/rocm/lib",
                           "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-multiple-definition", "-lpthread",
                           "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.split() == ["2", "1!", "2!", "4!"], out
