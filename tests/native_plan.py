"""The fp32 and bf16 planners of the GEMM headers as a host library, for tests
without a GPU: compiled from the headers themselves (host code only)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_08939_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
KINDS = ["HUGE", "WIDE", "TALL", "BIG", "SMALL", "NARROW", "MID", "DUO"]

SOURCE = r"""
#include <hip/hip_runtime.h>
#include "ard_gemm.hpp"
#include "ard_gemm_fast.hpp"
using namespace ard;
extern "C" {
void plan_f32(int M, int N, int K, int kb, int batch, long cap, int* out) {
  const FastPlan p = plan_fast_f32(M, N, K, kb, batch, cap), l = least_plan_f32(M, N, K, kb, batch, cap);
  out[0] = p.kind, out[1] = p.splits, out[2] = l.kind, out[3] = l.splits;
}
void plan_reg(int bf, int form, int M, int N, int K, long cap, int* out) {
  const FastPlan p = bf ? plan_any<bf16>(form, M, N, K, 1, 1, cap) : plan_any<float>(form, M, N, K, 1, 1, cap);
  out[0] = p.kind, out[1] = p.splits;
}
static GemmArgs product(int M, int N, int K) {
  GemmArgs g = {};
  g.M = M, g.N = N, g.K = K;
  return g;
}
int pair_f32(int B, int kin, int kout, long cap) {
  return fast_pair_ok<float>(product(kin, B, kout), product(kout, kin, B), cap);
}
}
"""


@pytest.fixture(scope="session")
def planner(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.hip", d / "libplan.so"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", f"-I{CSRC}",
                    str(src), "-o", str(lib)], check=True, capture_output=True)
    return Planner(ctypes.CDLL(str(lib)))


class Planner:
    ROOM = 1 << 60

    def __init__(self, lib):
        lib.plan_f32.argtypes = [ctypes.c_int] * 5 + [ctypes.c_long, ctypes.c_void_p]
        lib.plan_reg.argtypes = [ctypes.c_int] * 5 + [ctypes.c_long, ctypes.c_void_p]
        lib.pair_f32.argtypes = [ctypes.c_int] * 3 + [ctypes.c_long]
        self.lib = lib

    def f32(self, M, N, K, kb=1, batch=1, cap=ROOM):
        """(kind, splits) of the plan and of the one that sizes the least workspace."""
        out = (ctypes.c_int * 4)()
        self.lib.plan_f32(M, N, K, kb, batch, cap, out)
        return (KINDS[out[0]], out[1]), (KINDS[out[2]], out[3])

    def reg(self, dtype, form, M, N, K, cap=ROOM):
        """(kind, splits) on register loads; form 0 forward, 1 dX, 2 dW."""
        out = (ctypes.c_int * 2)()
        self.lib.plan_reg(int(dtype == "bf16"), form, M, N, K, cap, out)
        return KINDS[out[0]], out[1]

    def pair(self, B, kin, kout, cap=ROOM):
        """Whether an aligned fp32 layer's backward runs as one launch."""
        return bool(self.lib.pair_f32(B, kin, kout, cap))
