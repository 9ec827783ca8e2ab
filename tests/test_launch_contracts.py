"""Argument checks of the internal launchers that no ABI call reaches today:
they return hipErrorInvalidValue before any launch.  A small program is compiled
against the sources' headers and the built library and run on the CPU."""
import os
import subprocess

import pytest

from paper_1910_13444_amd import build

PROGRAM = r"""
#include <cstdio>
#include "pointwise.h"
using namespace pigan;
static NtArgs<float> nt(int pm) {
  NtArgs<float> a{};
  static float buf[64];
  a.X = buf; a.Wm = buf; a.aprev = buf; a.out_da = buf; a.ldx = a.ldw = a.ldo = 32;
  a.N = a.K = 32; a.pm = pm; a.seg = Seg{1, 0, 1}; a.a_seeds = 1;
  return a;
}
static CastSet<float> cast(int N, int K, int Kp, int pair, bool tr) {
  CastSet<float> c{};
  static float buf[64];
  c.src = buf; c.layers = 1; c.N = N; c.K = K; c.Kp = Kp; c.pair = pair; c.f = buf; c.fT = tr ? buf : nullptr;
  return c;
}
int main() {
  const CastSet<float> none{}, ok = cast(32, 20, 32, 1, true);
  const hipError_t got[] = {
    launch_gemm_nt<float>(EPI_BWD, 1, 0, nt(PM_SPLIT2), 1, nullptr),     // one row per stream: native products only
    launch_gemm_nt<float>(EPI_BWD, 1, 0, nt(PM_F64), 1, nullptr),
    launch_gemm_nt<float>(EPI_BWD, 1, 0, nt(3), 1, nullptr),             // no such product mode
    launch_cast_layers<float>(cast(32, 20, 24, 1, false), none, 1, nullptr),   // split copies: whole 16-element blocks
    launch_cast_layers<float>(cast(24, 32, 32, 1, true), none, 1, nullptr),
    launch_cast_layers<float>(ok, cast(32, 20, 24, 1, false), 1, nullptr)};
  int bad = 0;
  for (unsigned i = 0; i < sizeof got / sizeof got[0]; ++i)
    if (got[i] != hipErrorInvalidValue) { std::printf("call %u: %d\n", i, (int)got[i]); bad = 1; }
  return bad;
}
"""


def test_launchers_refuse_what_kernels_assume(tmp_path):
    if not os.path.exists(build.hipcc()) or not os.path.exists(build.LIB):
        pytest.skip("hipcc or the library is not available")
    src, exe = tmp_path / "contracts.cpp", str(tmp_path / "contracts")
    src.write_text(PROGRAM)
    r = subprocess.run([build.hipcc(), *build.common_flags(), "-xhip", str(src), "-xnone", build.LIB,
                        "-Wl,-rpath," + os.path.dirname(build.LIB), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60,
                       env={**os.environ, "HIP_VISIBLE_DEVICES": "-1", "ROCR_VISIBLE_DEVICES": "-1"})
    assert r.returncode == 0, r.stdout + r.stderr
