"""The choice of the decoder, on the CPU: launch_decode compiled for the host with
stub launchers, over every beam size, LM order, boosting and repeat scoring,
at the vocabularies around each line of the rule.  Whatever it picks must be
compiled: the general decoder holds beams of one chunk, and of several chunks
only in the forms that multi_chunk names and for at most 16 beams; two register
sets (beams above 64) exist up to 1024 tokens only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm/include"

PROGRAM = r"""
#include "ctcbeam_internal.h"
#include <cstdio>
using namespace ctcbeam;
static int g_lpt, g_class, g_rep;
namespace ctcbeam {
#define GENERAL(n)                                                                                      \
  hipError_t launch_lpt##n(const KernelParams&, hipStream_t) { g_lpt = n; g_class = g_rep = 0; return hipSuccess; } \
  hipError_t launch_lpt##n##_rep(const KernelParams&, hipStream_t) { g_lpt = n; g_class = 0; g_rep = 1; return hipSuccess; } \
  hipError_t launch_class_lpt##n(const KernelParams&, hipStream_t) { g_lpt = n; g_class = 1; g_rep = 0; return hipSuccess; }
GENERAL(1) GENERAL(2) GENERAL(4) GENERAL(8)
// (without the small-beam decoder, the others must serve its calls too)
bool small_beam_eligible(const KernelParams&) { return false; }
hipError_t launch_small(const KernelParams&, hipStream_t) { return hipSuccess; }
}
int main() {
  const int vs[] = {1, 2, 8, 9, 16, 17, 63, 64, 65, 512, 513, 1024, 1025, 1800, 1801, 2048, 2049, 2560, 2561, 3072, 3073, 4096};
  long calls = 0, general_multi = 0, bad = 0;
  static BtNode bt;
  static LmArc arc;
  static LmLevel lev;
  for (int V : vs)
    for (int K = 1; K <= (V <= 1024 ? kMaxK : kMaxKWideV); ++K)
      for (int nlev = -1; nlev <= 7; ++nlev)
        for (int b = 0; b < 2; ++b)
          for (int rep = 0; rep < 2; ++rep) {
            KernelParams p{};
            p.B = 1; p.V = V; p.K = K; p.flags = rep ? kFlagRepeatScore : 0;
            if (nlev >= 0) { p.lm_arcs = &arc; p.lm_states = &lev; p.lm_nlev = nlev; }
            if (b) p.bt_nodes = &bt;
            g_lpt = 0;
            launch_decode(p, nullptr);
            ++calls;
            bool ok = g_lpt > 0 && V <= 512 * g_lpt && (g_lpt == 1 || V > 256 * g_lpt);
            if (g_class) {
              ok = ok && (K <= 64 || V <= 1024) && K >= 3;
            } else {
              ok = ok && (K <= 16 / g_lpt || (K <= 16 && multi_chunk(g_lpt, nlev, b != 0)));
              ok = ok && g_rep == (rep && (nlev >= 0 || b));
              general_multi += K > 16 / g_lpt;
            }
            if (!ok && bad++ < 10) std::printf("V=%d K=%d nlev=%d bt=%d rep=%d -> lpt %d class %d\n", V, K, nlev, b, rep, g_lpt, g_class);
          }
  std::printf("calls %ld general_multi %ld bad %ld\n", calls, general_multi, bad);
  return bad != 0 || general_multi == 0;
}
"""


def test_every_choice_is_compiled(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(HIP, "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "dispatch.cpp", tmp_path / "dispatch"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{HIP}",
                    f"-I{os.path.join(ROOT, 'paper_2508_07315_amd', 'csrc')}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
