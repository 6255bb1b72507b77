"""The layout rule of the fused pseudogradient + update (plan_fused in
csrc/launch.hpp), compiled for the host, at sizes where the layouts it chooses
between were timed on an MI355X and differ by more than their noise."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_14563_amd", "csrc")
SRC = """
#include "launch.hpp"
extern "C" int plan(int full, long T, long d, long d_ff, long L, int grad_bf16, int adam, int state) {
  const fpo::FusedPlan p = fpo::plan_fused({full != 0, T, d, d_ff, L, grad_bf16 != 0, adam != 0, state != 0});
  return p.w3_first;
}
"""
W3_FIRST = 1


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([shutil.which("g++"), "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I",
                    os.path.join(rocm, "include"), "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True)
    f = C.CDLL(str(d / "plan.so")).plan
    f.argtypes = [C.c_int] + [C.c_long] * 4 + [C.c_int] * 3

    def call(full, T, d, d_ff, L, opt, staged=False):
        return f(full, T, d, d_ff, L, staged, opt == "adamw", opt != "plain")

    return call


# (T, d, d_ff, L, optimizer): us with the W3 launches first, last
@pytest.mark.parametrize("case,first,last", [((1024, 2048, 5504, 1, "adamw"), 333, 381),
                                             ((1024, 4096, 11008, 2, "adamw"), 2029, 2166),
                                             ((256, 4096, 11008, 1, "sgd"), 701, 781),
                                             ((512, 4096, 11008, 2, "sgd"), 1502, 1595),
                                             ((2048, 2048, 5504, 1, "sgd"), 386, 413),
                                             ((2048, 3072, 23040, 3, "adamw"), 5826, 5958),
                                             ((3000, 4096, 11008, 2, "sgd"), 3216, 3095),
                                             ((3000, 3072, 23040, 1, "adamw"), 3013, 2863),
                                             ((4096, 3072, 23040, 2, "sgd"), 5473, 5349),
                                             ((4096, 3072, 23040, 2, "adamw"), 5954, 5874)])
def test_full_mlp_order(plan, case, first, last):
    assert bool(plan(True, *case) & W3_FIRST) == (first < last)
