"""Products that no kernel computes are refused before anything is launched.  The struct behind the products is not part of the C interface, so
a small program built against the library makes the calls."""
import os
import subprocess

from paper_2507_10392_amd import build

PROGRAM = r"""
#include "kernels.h"
#include <cstdio>
using namespace zs;
// A product with GELU in its store, forward (act = 1) or backward (2), over addresses that are never read.
static Gemm product(int act, int M) {
  Gemm g;
  g.M = M; g.N = 2048; g.K = 512; g.transB = act == 2;
  g.A = (void*)4096; g.lda = g.K; g.B = (void*)8192; g.ldb = g.transB ? g.K : g.N; g.C = (void*)16384; g.ldc = g.N;
  g.act = act; g.act_z = (void*)32768;
  return g;
}
int main() {
  for (int act = 1; act <= 2; ++act) {
    for (DType dt : {BF16, F16})
      for (int M : {64, 256, 4096, 1 << 21}) {       // small tiles, few and many staged ones, cut into ranges of rows
        const Gemm g = product(act, M);
        printf("%d %d\n", (int)gemm(nullptr, dt, g, GEMM_AUTO), (int)(gemm_route(dt, g) == ROUTE_SIMPLE));
      }
    Gemm g = product(act, 256);
    g.transB ^= 1;                                   // fp32: the form that the other direction has
    g.ldb = g.transB ? g.K : g.N;
    printf("%d %d\n", (int)gemm(nullptr, F32, g, GEMM_AUTO), (int)(gemm_route(F32, g) == ROUTE_SIMPLE));
    printf("%d %d\n", (int)gemm(nullptr, F32, product(act, 256), GEMM_SIMPLE), (int)(gemm_route(F32, product(act, 256)) == ROUTE_F32));
  }
}
"""


def test_activation_outside_fp32_is_refused(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    src, exe = tmp_path / "refusals.hip", tmp_path / "refusals"
    src.write_text(PROGRAM)
    subprocess.run([build._hipcc(), *build.FLAGS, "-w", "-I", build.CSRC, str(src), f"-L{build.HERE}", "-l:libstage.so", f"-Wl,-rpath,{build.HERE}", "-o",
                    str(exe)], check=True, capture_output=True)
    no_gpu = dict(os.environ, HIP_VISIBLE_DEVICES="-1")              # a launch could only fail
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True, env=no_gpu).stdout.split("\n")[:-1]
    assert len(lines) == 20 and set(lines) == {"1 1"}, lines      # hipErrorInvalidValue
