"""Host check on the launch plan of the bf16 GEMM, asked from the built
library: a workspace that holds exactly the K slices the rule chose gives the
same count again. The update sums that many partial planes, so a launch that
took fewer would leave it planes that nobody wrote."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1809_02839_amd")
LIB = os.path.join(PKG, "libspectrain.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include "kernels.hpp"
using namespace spx;

// Slices of a convolution's filter gradient [c2][9 c] over `pix` pixels, by
// the rule and by a launch whose workspace holds that many partials.
int main() {
  const int channels[] = {24, 64, 72, 104, 128, 256, 328, 512}, batches[] = {1, 11, 32, 64, 113};
  long shapes = 0, split = 0, bad = 0;
  for (int c : channels)
    for (int c2 : channels)
      for (int b : batches)
        for (int h = 5; h <= 16; ++h)
          for (int w = h; w <= 16; w += 3) {
            const int pix = b * h * w, rule = gemm_bf16_split_rule(c2, 9 * c, pix, 1, 64u << 20);
            GemmDesc d;
            d.M = c2;
            d.N = 9 * c;
            d.K = pix;
            d.A.mode = OP_R_PLAIN;
            d.A.ld = c2;
            d.A.extent = static_cast<long>(pix) * c2;
            d.B.mode = OP_R_CONV_WGRAD;
            d.B.ld = c;
            d.B.extent = static_cast<long>(pix) * c;
            d.B.g = {b, h, w, c, 0};
            d.workspace = reinterpret_cast<float*>(256);   // an address only: nothing is launched
            d.workspace_bytes = static_cast<size_t>(rule) * c2 * 9 * c * 4;
            const int planned = gemm_bf16_splits(d);
            ++shapes;
            split += rule > 1;
            if (planned != rule && ++bad <= 10)
              std::printf("%d -> %d channels, %d x %d x %d: rule %d, launch %d\n", c, c2, b, h, w, rule, planned);
          }
  std::printf("shapes %ld split %ld bad %ld\n", shapes, split, bad);
  return split < 100 || bad != 0;
}
"""


def _run(program, tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(program)
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"), str(src), "-o", str(exe),
                    "-L", PKG, "-lspectrain", f"-Wl,-rpath,{PKG}"], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


needs_build = pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(HIPCC)),
                                 reason="needs the built library and hipcc")


@needs_build
def test_split_count_with_an_exactly_fitting_workspace(tmp_path):
    _run(PROGRAM, tmp_path)


# (M, N, K): slices alone, and beside another pass. Two blocks a CU, at least 12
# K steps a slice, at most 16; whole where 128 x 64 tiles fill three quarters of
# the slots (alone), or from 128 tiles on below 64 K steps (beside).
OCCUPANCY = {
    (960, 480, 1920): (2, 2), (960, 480, 4320): (5, 5), (480, 1920, 960): (1, 1), (2450, 512, 2048): (2, 2),
    (256, 1024, 12544): (16, 16), (256, 2304, 12544): (14, 14), (512, 4608, 2450): (3, 1), (24, 216, 2500): (3, 3),
    (6272, 512, 4608): (1, 2), (19200, 64, 1600): (2, 1), (12544, 1024, 256): (1, 1),
}


@needs_build
def test_occupancy_slices(tmp_path):
    calls = "".join(f'std::printf("%d %d\\n", gemm_bf16_split_rule({m}, {n}, {k}, 1, 64u << 20, SPLIT_OCCUPANCY), '
                    f'gemm_bf16_split_rule({m}, {n}, {k}, 1, 64u << 20, SPLIT_OCCUPANCY_SHARED));\n'
                    for m, n, k in OCCUPANCY)
    out = _run('#include <cstdio>\n#include "kernels.hpp"\nusing namespace spx;\nint main() {\n' + calls + "}\n",
               tmp_path)
    assert [tuple(map(int, l.split())) for l in out.splitlines()] == list(OCCUPANCY.values())
