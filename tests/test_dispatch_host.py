"""Host checks on the dispatch rules, asked from the built library.

bf16 GEMM: a workspace that holds exactly the K slices the rule chose gives the
same count again (the update sums that many partial planes, so a launch that
took fewer would leave it planes that nobody wrote), and bottleneck stages take
the slices that fill the CUs. LSTM, attention and float32 GEMM: the rules take
the faster path where both were measured."""
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


# us of a one-layer step (T = 16, forward, backward and update), one fused
# launch per time step against a GEMM and a cell launch, by (H, B).
LSTM_TIMES = {
    (8, 4096): (226, 458), (8, 16384): (559, 703), (64, 1024): (205, 470), (64, 4096): (463, 561),
    (64, 16384): (1624, 1210), (128, 4096): (869, 748), (256, 256): (230, 511), (256, 1024): (533, 638),
    (256, 1536): (780, 721), (512, 64): (254, 524), (512, 320): (549, 644), (512, 512): (732, 743),
    (512, 640): (903, 809), (776, 224): (699, 773), (1024, 8): (300, 484), (1024, 64): (390, 552),
    (1024, 128): (644, 758), (1024, 160): (856, 816), (1024, 256): (1128, 939), (1032, 100): (668, 777),
    (1280, 64): (718, 672), (1280, 80): (752, 713), (1536, 32): (567, 644), (1536, 48): (843, 709),
    (1536, 96): (1196, 849), (2048, 16): (705, 764), (2048, 32): (800, 810), (2048, 64): (1239, 944),
    (2560, 8): (943, 993), (2560, 32): (1522, 1164), (3072, 64): (2590, 1693), (4096, 32): (2771, 2175),
}


@needs_build
def test_lstm_rule_takes_the_faster_path(tmp_path):
    calls = "".join(f'std::printf("%d\\n", int(lstm_step_supported({b}, {h})));\n' for h, b in LSTM_TIMES)
    calls += 'std::printf("%d %d %d %d\\n", int(lstm_step_supported(0, 64)), int(lstm_step_supported(4, 0)), ' \
             'int(lstm_step_supported(4, 68)), int(lstm_step_supported(1 << 30, 8)));\n'
    *got, refused = _run('#include <cstdio>\n#include "kernels.hpp"\nusing namespace spx;\nint main() {\n' + calls +
                         "}\n", tmp_path).splitlines()
    assert refused == "0 0 0 0"
    slower = {hb: (t[1 - int(g)], t[int(g)]) for (hb, t), g in zip(LSTM_TIMES.items(), got)
              if (t[0] if int(g) else t[1]) > 1.07 * min(t)}
    assert not slower, slower


# us of a float32 product X W^T on the short and on the tile kernel (with its
# reduction), by (M, N, K).
F32_TIMES = {
    (32, 10, 128): (6.5, 9.9), (32, 10, 512): (8.9, 11.4), (32, 10, 2048): (20.1, 13.0), (32, 10, 16384): (124, 17.7),
    (32, 10, 262144): (1970, 110), (64, 64, 256): (8.0, 11.4), (64, 64, 4096): (40.3, 14.3),
    (128, 64, 512): (10.5, 11.8), (128, 128, 2048): (23.5, 13.9), (256, 128, 8192): (76.1, 20.1),
    (256, 256, 512): (10.0, 12.6), (256, 256, 4096): (42.2, 19.0), (512, 256, 256): (8.4, 11.7),
    (512, 256, 2048): (25.8, 19.1),
}


@needs_build
def test_float32_rule_takes_the_faster_kernel(tmp_path):
    calls = "".join(f"std::puts(name({m}, {n}, {k}));\n" for m, n, k in F32_TIMES)
    got = _run("""#include <cstdio>
#include "kernels.hpp"
using namespace spx;
const char* name(int m, int n, int k) {
  GemmDesc d;
  d.M = m;
  d.N = n;
  d.K = k;
  d.A.ld = d.B.ld = k;
  d.workspace = reinterpret_cast<float*>(256);   // an address only: nothing is launched
  d.workspace_bytes = 8u << 20;
  return gemm_f32_kernel_name(d);
}
int main() {
""" + calls + "}\n", tmp_path).split("\n")
    slower = {p: t for (p, t), g in zip(F32_TIMES.items(), got)
              if t[0 if g.startswith("gemm_f32_short") else 1] > 1.05 * min(t)}
    assert not slower, slower


# us of an encoder layer's step, score tiles against batched GEMMs, by (batch, S,
# heads) at head dimension 64.
ATTENTION_TIMES = {
    (1, 512, 1): (271, 278), (2, 640, 1): (268, 308), (8, 640, 1): (278, 298), (1, 768, 4): (290, 311),
    (1, 1024, 1): (325, 288), (1, 1024, 4): (331, 299), (1, 1024, 8): (363, 345), (12, 1024, 1): (349, 367),
    (16, 1024, 1): (354, 400), (1, 2048, 1): (466, 327), (5, 2048, 1): (486, 457), (6, 2048, 1): (490, 504),
    (1, 2048, 8): (511, 613), (1, 4096, 1): (758, 417), (2, 4096, 1): (765, 576), (3, 4096, 1): (775, 811),
    (1, 8192, 1): (1337, 1089), (1, 12288, 1): (1921, 2239), (24, 328, 8): (433, 600),
}


@needs_build
def test_attention_rule_takes_the_faster_path(tmp_path):
    calls = "".join(f'std::printf("%d\\n", int(attention_long_preferred({b}, {s}, {h})));\n' for b, s, h in ATTENTION_TIMES)
    got = _run('#include <cstdio>\n#include "kernels.hpp"\nusing namespace spx;\nint main() {\n' + calls + "}\n",
               tmp_path).split()
    slower = {c: t for (c, t), g in zip(ATTENTION_TIMES.items(), got) if t[1 - int(g)] > 1.02 * min(t)}
    assert not slower, slower
