"""The build refuses a kernel whose requested loop unrolling the compiler drops."""
import subprocess

import pytest

from paper_2207_08867_amd import build

# A loop of the product kernels' form (a run-time trip count, two steps an iteration asked
# for) around an asm statement, which counts as convergent: it stays rolled.
ROLLED_LOOP = r"""
#include <hip/hip_runtime.h>
__global__ void k(const _Float16 *a, _Float16 *c, int n) {
  _Float16 s = 0;
#pragma unroll 2
  for (int i = 0; i < n; ++i) {
    _Float16 e;
    asm("v_pk_fma_f16 %0, %1, %2, %3" : "=v"(e) : "v"(a[i]), "v"(s), "v"(s));
    s = e;
  }
  c[threadIdx.x] = s;
}
"""


def test_a_dropped_unroll_fails_the_build(tmp_path):
    src = tmp_path / "k.hip"
    src.write_text(ROLLED_LOOP)
    r = subprocess.run([build.HIPCC, *build.CFLAGS, "-c", str(src), "-o", str(tmp_path / "k.o")], capture_output=True,
                       text=True)
    assert r.returncode != 0 and "loop not unrolled" in r.stderr


@pytest.mark.parametrize("src", build.SOURCES)
def test_only_the_exponentials_may_keep_rolled_loops(src):
    assert (src in build.ROLLED) == (src in ("elementwise.hip", "exp64.hip"))
