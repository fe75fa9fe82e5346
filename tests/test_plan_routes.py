"""The plan's choice of a tail batch's scan against the forms' measured times.

gdn_plan.cpp is plain C++, so it is built here with the host compiler behind a
one-function shim.  Each row is a batch that both forms were timed on (MI355X,
whole calls, us): the plan has to take the faster one.  A CPU test: where the
two are within a few per cent of each other there is no row.
"""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2608_30310_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "gdn_plan.h"
extern "C" int tail_route(const gdn_shape* s, const int32_t* cu) {
  gdn::Plan p;
  std::string err;
  if (gdn::make_plan(s, cu, false, &p, &err) != GDN_OK) return -1;
  return static_cast<int>(gdn::tail_scan(*s, cu, p));
}
"""
ROUNDS, WIDE, HEAD = 0, 1, 2


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "shim.cpp", d / "libplan.so"
    src.write_text(SHIM)
    csrc = os.path.join(ROOT, "paper_2608_30310_amd", "csrc")
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    "-o", str(lib), str(src), os.path.join(csrc, "gdn_plan.cpp")], check=True)
    fn = ctypes.CDLL(str(lib)).tail_route

    def of(hk, hv, dk, dv, chunks, dtype):
        cu = [0]
        for c in chunks:
            cu.append(cu[-1] + 64 * c)
        s = binding.GDNShape(len(chunks), hk, hv, dk, dv, dtype, 1.0)
        return fn(ctypes.byref(s), (ctypes.c_int32 * len(cu))(*cu))
    return of


# hk, hv, dk, dv, chunks per sequence, us in 64-column rounds, us with a head per workgroup
F32_BATCHES = [
    (16, 32, 128, 128, [2] * 5, 25.9, 22.8),
    (16, 32, 128, 128, [4] + [1] * 4, 22.5, 29.4),
    (16, 32, 128, 128, [7] * 12, 86.3, 94.9),
    (16, 32, 128, 128, [1] * 16, 38.2, 33.6),
    (16, 32, 128, 128, [7] + [1] * 35, 71.5, 60.4),
    (16, 32, 64, 128, [4] * 9, 40.4, 44.8),
    (16, 32, 64, 128, [4] + [1] * 35, 58.2, 45.4),
    (16, 32, 64, 128, [1] * 24, 41.3, 35.7),
    (4, 4, 128, 128, [7] + [1] * 39, 29.9, 41.9),
    (4, 4, 128, 128, [1] * 300, 91.7, 82.7),
    (1, 1, 64, 128, [7] + [1] * 199, 24.3, 31.9),
    (1, 1, 64, 128, [7] * 600, 108.8, 115.8),
]


@pytest.mark.parametrize("hk,hv,dk,dv,chunks,rounds,head", F32_BATCHES)
def test_fp32_tail_batches(route, hk, hv, dk, dv, chunks, rounds, head):
    assert route(hk, hv, dk, dv, chunks, binding.GDN_F32) == (ROUNDS if rounds < head else HEAD)


def test_fp32_tail_batches_with_one_form(route):
    # 64-column workgroups that fit at once, and heads of one such workgroup
    assert route(16, 32, 128, 128, [1] * 4, binding.GDN_F32) == ROUNDS
    assert route(16, 32, 128, 64, [1] * 36, binding.GDN_F32) == ROUNDS
    assert route(16, 32, 128, 128, [], binding.GDN_F32) == ROUNDS
    assert route(65535, 65535, 128, 128, [1], binding.GDN_F32) in (ROUNDS, HEAD)
