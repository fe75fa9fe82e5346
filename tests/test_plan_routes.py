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


# hk, hv, dk, dv, chunks per sequence, us in 64-column rounds, us in the wide scan
BF16_BATCHES = [
    (16, 32, 128, 128, [13] * 5, 59.9, 54.2),
    (16, 32, 128, 128, [52] + [3] * 4, 87.7, 144.5),
    (16, 32, 128, 128, [2, 4, 2, 4, 2, 4, 2, 4, 2], 31.6, 28.0),
    (16, 32, 128, 128, [13] * 12, 92.0, 83.9),
    (16, 32, 128, 128, [52] + [3] * 35, 121.8, 183.5),
    (1, 140, 128, 128, [13, 7], 81.9, 74.0),
    (16, 32, 64, 128, [52] + [3] * 4, 62.3, 109.6),
    (16, 32, 64, 128, [13] * 8, 49.8, 48.6),
    (16, 32, 128, 64, [13] * 12, 70.4, 67.1),
    (16, 32, 128, 64, [52] + [3] * 11, 92.8, 147.3),
    (16, 32, 64, 64, [13] * 9, 51.2, 58.3),
    (16, 32, 64, 64, [13] * 16, 64.4, 71.1),
    (16, 32, 64, 64, [13] * 24, 91.4, 101.0),
    (16, 32, 64, 64, [7] * 17, 51.4, 56.2),
    (4, 4, 64, 64, [13] * 128, 65.7, 72.1),
    (2, 300, 64, 64, [7], 37.5, 40.5),
    # beyond 256 sequences there is no order
    (1, 1, 128, 128, [13] * 300, 86.1, 78.4),
    (1, 1, 128, 128, [52] + [3] * 299, 84.9, 145.8),
    (1, 1, 128, 128, list(range(1, 27)) * 12, 103.4, 120.5),
    (1, 1, 64, 64, [13] * 300, 54.1, 60.8),
    (1, 1, 64, 64, [52] + [3] * 599, 70.1, 114.9),
    (1, 1, 64, 64, [13] * 600, 83.3, 78.8),
    (4, 4, 64, 64, [52] + [3] * 299, 77.5, 125.0),
]


@pytest.mark.parametrize("hk,hv,dk,dv,chunks,rounds,wide", BF16_BATCHES)
def test_bf16_tail_batches(route, hk, hv, dk, dv, chunks, rounds, wide):
    assert route(hk, hv, dk, dv, chunks, binding.GDN_BF16) == (ROUNDS if rounds < wide else WIDE)
