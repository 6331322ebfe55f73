"""find_kernel on stub tables: every entry is found, everything else is not, and
building the table allocates nothing (it happens inside a C entry point)."""
import os
import subprocess

import pytest

from paper_2608_25203_amd import build

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <new>
#include "zk_kernels.hpp"
static int news = 0;
void *operator new(size_t n) { ++news; return std::malloc(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
namespace zk {
static KernelEntry tab[4][300];
extern const KernelEntry *const row_kernels_f64[] = {tab[0], nullptr}, *const row_kernels_f32[] = {tab[1], nullptr},
                                *const col_kernels_f64[] = {tab[2], nullptr}, *const col_kernels_f32[] = {tab[3], nullptr};
}
using namespace zk;
int main() {
  static char mark[4][300];
  for (int t = 0; t < 4; ++t)
    for (int i = 0; i < 250; ++i) tab[t][i] = {1 + (i * 37) % 1024, 2 + i % 14, i % 2 == 0, i % 5, &mark[t][i]};
  int bad = 0;
  news = 0;  // the runtime may have allocated before main
  for (int t = 0; t < 4; ++t)
    for (int i = 0; i < 250; ++i) {
      const KernelEntry &k = tab[t][i];
      bad += find_kernel(t < 2, t % 2 == 0, k.form, k.T, k.E, k.pad) != k.fn;
      bad += find_kernel(t < 2, t % 2 == 0, k.form, k.T, 1, k.pad) != nullptr;
    }
  std::printf("%d %d", bad, news);
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_lookup_allocates_nothing(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    inc = ["-I", build.CSRC, "-I", os.path.join(build.ROOT, "include")]
    objs = []
    for src in (str(tmp_path / "main.cpp"), os.path.join(build.CSRC, "zk_launch.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        subprocess.run([build.HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-x", "hip", *inc, "-c", src,
                        "-o", objs[-1]], check=True)
    subprocess.run([build.HIPCC, *objs, "-o", str(tmp_path / "lookup")], check=True)
    out = subprocess.run([str(tmp_path / "lookup")], check=True, capture_output=True, text=True).stdout
    assert out == "0 0"
