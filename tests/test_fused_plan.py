"""The layout rule of the fused pseudogradient + update (plan_fused in
csrc/launch.hpp), compiled for the host, at sizes where the layouts it chooses
between were timed on an MI355X and differ by more than their noise; and the grid
of a launch of quarters (quarter_grid)."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_14563_amd", "csrc")
SRC = """
#include "launch.hpp"
extern "C" int plan(int full, long T, long d, long d_ff, long L, int grad_bf16, int adam, int state, int ref) {
  const fpo::FusedPlan p = fpo::plan_fused({full != 0, T, d, d_ff, L, grad_bf16 != 0, adam != 0, state != 0, ref != 0});
  return p.w3_first | p.overlap << 1 | p.two_per_cu << 2;
}
extern "C" int quarters(long M, long N, long mats, long nbig) { return fpo::quarter_grid(M, N, mats, nbig); }
"""
W3_FIRST, OVERLAP, TWO_PER_CU = 1, 2, 4


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([shutil.which("g++"), "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I",
                    os.path.join(rocm, "include"), "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True)
    return C.CDLL(str(d / "plan.so"))


@pytest.fixture(scope="module")
def plan(host):
    f = host.plan
    f.argtypes = [C.c_int] + [C.c_long] * 4 + [C.c_int] * 4

    def call(full, T, d, d_ff, L, opt, staged=False, ref=False):
        return f(full, T, d, d_ff, L, staged, opt == "adamw", opt != "plain", ref)

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


# (T, d, d_ff, L, optimizer, staged in bf16): us overlapped, batched
@pytest.mark.parametrize("case,overlapped,batched", [((1024, 4096, 12288, 6, "sgd", False), 1519, 1805),
                                                     ((1024, 4096, 11008, 4, "sgd", False), 991, 1107),
                                                     ((1024, 4096, 11008, 8, "adamw", False), 2621, 2772),
                                                     ((1024, 4096, 11008, 8, "sgd", True), 1732, 1999),
                                                     ((512, 4096, 11008, 8, "sgd", False), 1874, 1958),
                                                     ((2048, 2048, 5504, 8, "adamw", False), 785, 864),
                                                     ((2500, 1536, 8960, 3, "adamw", False), 392, 418),
                                                     ((1024, 1536, 8960, 16, "sgd", False), 1227, 1360),
                                                     ((1024, 4096, 12288, 6, "plain", False), 1166, 1375),
                                                     ((700, 3072, 23040, 16, "sgd", False), 5758, 6504),
                                                     ((4096, 1536, 8960, 3, "adamw", True), 467, 507),
                                                     ((300, 4096, 11008, 8, "sgd", True), 1545, 1654),
                                                     ((2048, 4096, 11008, 8, "sgd", True), 2177, 2589),
                                                     ((300, 4096, 11008, 2, "sgd", True), 419, 404),
                                                     ((512, 4096, 11008, 8, "adamw", True), 2374, 2272),
                                                     ((512, 3744, 9048, 5, "plain", True), 618, 594),
                                                     ((128, 3072, 23040, 6, "plain", True), 1275, 1197),
                                                     ((608, 2912, 10808, 4, "adamw", True), 894, 834),
                                                     ((1536, 2048, 5504, 4, "sgd", False), 336, 308),
                                                     ((1800, 1536, 8960, 2, "adamw", False), 264, 251),
                                                     ((2944, 2048, 5504, 8, "sgd", False), 884, 858),
                                                     ((4096, 1536, 8960, 6, "plain", False), 798, 760),
                                                     ((1024, 2048, 5504, 4, "sgd", True), 280, 264),
                                                     # partly filled waves: 288, 156, 290 tiles a layer
                                                     ((1792, 1840, 9088, 3, "sgd", False), 447, 391),
                                                     ((6020, 1472, 6584, 5, "adamw", False), 1010, 813),
                                                     ((2675, 2472, 7176, 4, "sgd", True), 718, 606)])
def test_w3_overlap(plan, case, overlapped, batched):
    assert bool(plan(False, *case) & OVERLAP) == (overlapped < batched)


def test_one_layer_of_w3_is_batched(plan):
    assert not plan(False, 4096, 4096, 12288, 1, "sgd") & OVERLAP


# (T, d, d_ff, L, optimizer): us overlapped (the better order), batched
@pytest.mark.parametrize("case,overlapped,batched", [((256, 2048, 5504, 6, "sgd"), 1253, 1394),
                                                     ((256, 4096, 11008, 1, "sgd"), 701, 763),
                                                     ((512, 4096, 11008, 1, "sgd"), 782, 852),
                                                     ((1024, 2048, 5504, 1, "adamw"), 333, 353),
                                                     ((2048, 4096, 11008, 6, "sgd"), 6531, 7769),
                                                     ((1021, 1320, 6440, 5, "sgd"), 1242, 1386),
                                                     ((4096, 3072, 23040, 2, "adamw"), 5874, 6489),
                                                     ((824, 1248, 5432, 3, "adamw"), 587, 707),
                                                     ((915, 2088, 6152, 12, "plain"), 3089, 3608),
                                                     ((966, 1808, 5272, 2, "sgd"), 487, 566),
                                                     ((512, 1024, 4096, 2, "sgd"), 259, 231),
                                                     ((512, 2048, 5504, 1, "sgd"), 251, 237),
                                                     ((2048, 1024, 4096, 6, "sgd"), 1182, 1028),
                                                     ((4096, 1024, 4096, 3, "adamw"), 943, 797)])
def test_full_mlp_overlap(plan, case, overlapped, batched):
    assert bool(plan(True, *case) & OVERLAP) == (overlapped < batched)


# (T, d, d_ff, L, optimizer, staged, against references): us with two update workgroups a CU, one
@pytest.mark.parametrize("case,two,one", [((1024, 4096, 11008, 8, "sgd", True), 1732, 2035),
                                          ((2048, 4096, 11008, 8, "sgd", True), 2177, 2340),
                                          ((700, 4096, 12288, 6, "sgd", False), 1509, 1568),
                                          ((1024, 4096, 12288, 16, "sgd", False), 3917, 4331),
                                          ((1024, 8192, 28672, 6, "plain", False), 5624, 5946),
                                          ((1800, 3072, 23040, 16, "sgd", False), 7379, 6956),
                                          ((1024, 8192, 28672, 6, "sgd", False), 7756, 7536),
                                          ((4096, 3072, 23040, 6, "sgd", False), 4246, 4162),
                                          ((2048, 4096, 11008, 6, "sgd", True, True), 2147, 2020),
                                          ((700, 4096, 12288, 6, "sgd", False, True), 1844, 1798)])
def test_update_workgroups_per_cu(plan, case, two, one):
    p = plan(False, *case)
    assert p & OVERLAP and bool(p & TWO_PER_CU) == (two < one)


@pytest.mark.parametrize("M,N,mats,nbig,want", [(64, 4096, 8, 0, 8 * 32), (130, 8, 1, 0, 2), (1, 1, 3, 0, 3),
                                                (111, 16496, 2, 0, 2 * 129), (256, 512, 2, 0, 16),
                                                (2048, 2816, 3, 256, 4 * 8), (300, 300, 1, 1, 12)])
def test_quarters_have_a_workgroup_each(host, M, N, mats, nbig, want):
    """A list that goes as quarters altogether has one workgroup per 128 x 128 tile
    inside its matrices; the tail of a list, four per 256 x 256 tile left."""
    f = host.quarters
    f.argtypes = [C.c_long] * 4
    assert f(M, N, mats, nbig) == want
