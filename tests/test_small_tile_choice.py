"""The products of the tests of the small tiles do run on the tiles that those tests are about.  The choice is not part of the C interface, so
a small program built against the library asks for it; nothing is launched."""
import os
import subprocess

from paper_2507_10392_amd import build
import test_rows_through_lds as lds
import test_small_products_both_ways as ways

PROGRAM = r"""
#include "kernels.h"
#include <cstdio>
using namespace zs;
int main() {
  int dt, tb, glu, M, N, K; long long ldb;
  while (scanf("%d %d %d %d %d %d %lld", &dt, &tb, &glu, &M, &N, &K, &ldb) == 7) {
    Gemm g;
    g.M = M; g.N = N; g.K = K; g.transB = tb;
    g.A = (void*)4096; g.lda = K; g.B = (void*)8192; g.ldb = ldb; g.C = (void*)16384; g.ldc = N;
    if (glu) { g.glu = 1; g.sB = (long long)K * N; g.gu = (void*)32768; g.gu_ld = 2 * N; g.gu_up = N; }
    const GemmRoute r = gemm_route((DType)dt, g);
    printf("%d\n", r == ROUTE_SMALL ? gemm_small_tile(g) : r == ROUTE_STAGED ? 128 : -1);
  }
}
"""


def test_products_of_the_tests_take_the_tiles_they_name(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    src, exe = tmp_path / "tiles.hip", tmp_path / "tiles"
    src.write_text(PROGRAM)
    subprocess.run([build._hipcc(), *build.FLAGS, "-w", "-I", build.CSRC, str(src), f"-L{build.HERE}", "-l:libstage.so", f"-Wl,-rpath,{build.HERE}", "-o",
                    str(exe)], check=True, capture_output=True)
    asked = []
    for dt in (1, 2):
        asked += [((dt, 1, 0, M, N, K, K), 64 if M == 1000 else 32) for d, M, N in lds.OUTPUTS if d == dt for K in lds.DEPTHS]
        asked += [((dt, 1, 0, M, N, K, K), 64 if M == 1000 else 32) for M, N in ways.GRADIENTS for K in ways.DEPTHS]
        asked += [((dt, 0, glu, M, N, K, N), 32) for M, N, K in ways.FORWARDS for glu in (0, 1)]
        asked += [((dt, 0, 0, ways.FAR_M, ways.FAR_N, ways.FAR_K, ldb), tile) for ldb, tile in ways.FAR]
    no_gpu = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, env=no_gpu, input="\n".join(" ".join(map(str, a)) for a, _ in asked))
    got = [int(x) for x in out.stdout.split()]
    assert got == [t for _, t in asked], [(a, t, x) for (a, t), x in zip(asked, got) if t != x]
