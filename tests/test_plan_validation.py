"""validate_plan refuses plans that the column kernels cannot run: each case
breaks one output of a valid plan."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_25203_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "zk_plan.hpp"
using namespace zk;
// argv[1]: what to break; prints validate_plan's answer
int main(int, char **argv) {
  PlanParams pp{};
  pp.nx = pp.ny = 64;
  pp.M = 3;
  pp.Lx = pp.Ly = 1.0;
  pp.g = 9.81;
  pp.eps = 1.0;
  pp.taper = pp.filt = true;
  Plan p = build_plan(pp, 0.01);
  ColOut &layer = p.outs[p.tasks[p.depth_chunk[2][0].first + 1].o0];
  const char *what = argv[1];
  if (!strcmp(what, "couple only")) layer.lift_sym &= ~(SYM_LAYER_C | SYM_LAYER_S);
  if (!strcmp(what, "no couple")) layer.lift_sym &= ~SYM_COUPLE;
  if (!strcmp(what, "both factors")) layer.lift_sym |= SYM_LAYER_C | SYM_LAYER_S;
  if (!strcmp(what, "keep in folds"))
    for (auto &l : p.step_body_lift[0])
      if (l.d2 == kMaxFolds)
        for (int k = l.first; k < l.first + l.count; ++k) p.outs[p.tasks[k].o0].keep = p.outs[p.tasks[k].o0].dst_base >= 0;
  if (!strcmp(what, "step_lift")) {
    std::printf("%d", (int)p.step_lift[0].size());
    pp.separate_lifts = true;
    std::printf(" %d", (int)build_plan(pp, 0.01).step_lift[0].size());
    return 0;
  }
  std::printf("%s", validate_plan(p, 3 * pp.ny / 2, pp.ny).c_str());
  return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(d / "main.cpp"),
                    os.path.join(CSRC, "zk_plan.cpp"), "-o", str(d / "plan")], check=True)
    return str(d / "plan")


@pytest.mark.parametrize("what,answer", [("nothing", ""), ("couple only", "lift_sym without its layer factor"),
                                         ("no couple", "lift_sym without its layer factor"),
                                         ("both factors", "lift_sym without its layer factor"),
                                         ("keep in folds", "kept output in a fold team launch")])
def test_broken_plan_is_refused(exe, what, answer):
    assert subprocess.run([exe, what], check=True, capture_output=True, text=True).stdout == answer


def test_separate_lifts_are_planned_on_request_only(exe):
    """The library's steps lift in their last launch; no call runs step_lift."""
    assert subprocess.run([exe, "step_lift"], check=True, capture_output=True, text=True).stdout == "0 1"


@pytest.mark.skipif(not os.path.exists(os.path.join(ROOT, "paper_2608_25203_amd", "libzk.so")), reason="libzk.so not built")
def test_options_set_to_their_value_keep_the_layout():
    """zk_set_option with the value an option has re-plans nothing: a hundred such
    calls take less than ten that change it (each of those builds a plan)."""
    import time

    from paper_2608_25203_amd import zk

    c = zk.zk_create(128, 96, 1.0, 1.0, 1.0, 9.81, 5)
    n = zk.zk_workspace_bytes(c)
    t0 = time.perf_counter()
    for _ in range(100):
        zk.zk_set_option(c, zk.ZK_OPT_PRECISION, 64)
    t1 = time.perf_counter()
    assert zk.zk_workspace_bytes(c) == n
    for k in range(10):
        zk.zk_set_option(c, zk.ZK_OPT_PRECISION, 64 if k % 2 else 32)
    t2 = time.perf_counter()
    assert zk.zk_workspace_bytes(c) == n
    zk.zk_destroy(c)
    assert t1 - t0 < t2 - t1
