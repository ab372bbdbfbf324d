"""The rules that pick a projection's launches (csrc/gemm_plan.h), compiled for the CPU."""
import ctypes as C
import os
import subprocess

import pytest

import test_gpu_project as gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2601_17818_amd", "csrc", "gemm_plan.h")

WRAPPER = """
#include "%s"
using namespace vitcop;
extern "C" {
int splitk(int M, int N, int K, int* o) {
    const SplitKPlan p = splitk_plan(M, N, K);
    o[0] = p.bm; o[1] = p.bn;
    return p.splits;
}
int most_slices(int M, int N, int K) { return splitk_most(M, N, K); }
int whole_tile(int M, int N, int K, int* o) {
    const TileShape& t = kTiles[choose_tile(M, N, K, false, 768)];
    o[0] = t.bm; o[1] = t.bn;
    return 0;
}
int qkv(int M, int qd, int kd, int d, int K, int* o) {
    const SplitKPlan p = qkv_plan(M, qd, kd, K);
    o[0] = p.bm; o[1] = p.bn;
    return qkv_path(M, qd, kd, d, K);
}
int gated_columns(int M, int F, int K) { return skinny_gated_columns(skinny_plan(M, 2 * F, K), M, F, K); }
int streams(int qd, int kd, int d, int D) { return stream_samples(qd, kd, d, D); }
int direct(int N) { return skinny_direct(N, false); }
int few_rows(int M, int N, int K, int* o) {
    const SkinnyPlan p = skinny_plan(M, N, K);
    o[0] = skinny_rows(M); o[1] = p.cols;
    return p.slices;
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(WRAPPER % HEADER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", str(d / "plan.so"), str(d / "plan.cpp")], check=True)
    return C.CDLL(str(d / "plan.so"))


def picked(plan, M, N, K):
    """(rows, columns, slices) of the tiles of a launch of 257 rows or more; whole tiles have 1 slice."""
    o = (C.c_int * 2)()
    slices = plan.splitk(M, N, K, o)
    if slices == 0:
        plan.whole_tile(M, N, K, o)
    return o[0], o[1], max(slices, 1)


@pytest.mark.parametrize("M,N,K,least,most", [
    # narrow outputs: each further slice costs the reduction more than it saves (21 us in 14 slices, 18 in 4 to 8)
    (576, 512, 3584, 1, 8), (1000, 512, 3584, 1, 8), (480, 768, 3072, 1, 8), (700, 1024, 2816, 1, 8),
    # one round of whole tiles over a long k takes a fifth to two fifths longer than slices of large tiles
    (640, 3584, 3584, 2, 3), (1000, 4096, 11008, 2, 4), (1024, 3584, 14336, 3, 4), (800, 5120, 13824, 3, 3),
    # tiles full of rows take longer than ones that end in padding, which is not loaded (whole tiles 56 and 21 us)
    (640, 5120, 5120, 2, 3), (640, 512, 3584, 4, 8),
    # few columns, short k: the narrow whole tiles need no reduction (12.5 us against 19 in the best number of slices)
    (320, 2048, 2048, 1, 1), (257, 1024, 1024, 1, 1)])
def test_slices_are_priced(plan, M, N, K, least, most):
    assert least <= picked(plan, M, N, K)[2] <= most


def test_slices_fit_the_scratch_that_callers_provide(plan):
    for M in range(1, 1700):
        for N, K in ((512, 3584), (1024, 1024), (4096, 4096), (5120, 5120), (9216, 8192), (3584, 14336), (272, 4128)):
            slices = picked(plan, M, N, K)[2]
            assert slices == 1 or (256 < M <= 1536 and slices <= plan.most_slices(M, N, K))


@pytest.mark.parametrize("M,N,K", [(5, 1024, 1024), (8, 1024, 1024), (8, 256, 1024), (16, 512, 1024)])
def test_slices_of_few_rows_are_priced(plan, M, N, K):
    """Small outputs over a short k: 9 us in 16 slices, 7.5 in 4 to 8."""
    assert plan.few_rows(M, N, K, (C.c_int * 2)()) <= 8


@pytest.mark.parametrize("M,N,K", gpu.LONG_SLICES)
def test_long_slices_are_long(plan, M, N, K):
    slices = plan.few_rows(M, N, K, (C.c_int * 2)()) if M <= 256 else picked(plan, M, N, K)[2]
    assert (K + 63) // 64 // slices >= 32
    rows = (M + 31) // 32 * 32 if M <= 256 else picked(plan, M, N, K)[0]
    assert (M <= 2 * rows) == ((M, N, K) in gpu.SPREAD_SLICES)


def test_slices_of_tall_launches(plan):
    """1025 to 1536 rows: within the scratch, on the tiles that the GPU tests reach, none above."""
    reached = {t[:2] for t in (picked(plan, *s) for s in gpu.SPLIT_K) if t[2] > 1}
    cut = 0
    for M in list(range(1025, 1600, 5)) + [1536, 1537, 3000]:
        for N, K in ((512, 3584), (1024, 1024), (2048, 5632), (4096, 4096), (5120, 5120), (3584, 14336), (272, 4128)):
            *tile, slices = picked(plan, M, N, K)
            if M > 1536:
                assert slices == 1
            elif slices > 1:
                assert slices <= plan.most_slices(M, N, K) and tuple(tile) in reached
                cut += 1
    assert cut > 50
    for M, N, K in gpu.SPLIT_TALL:
        assert picked(plan, M, N, K)[2] > 1


@pytest.mark.parametrize("D,Hq,Hkv,d,samples", [
    (4096, 32, 32, 128, 3), (3584, 28, 4, 128, 3), (2048, 16, 16, 128, 3), (1024, 16, 4, 64, 3), (4160, 24, 6, 128, 3),
    # widths of K and V that are no whole groups of 128 columns: the matrix cores would take three launches and the rotary one
    (1024, 16, 1, 64, 4), (2048, 32, 1, 64, 4), (2048, 24, 3, 64, 4), (4096, 64, 1, 64, 4)])
def test_four_decoding_samples_take_the_faster_way(plan, D, Hq, Hkv, d, samples):
    assert plan.streams(Hq * d, Hkv * d, d, D) == samples


def sliced(plan, M, N, K):
    """The tile of a launch of one matrix or a pair that is cut over k, or nothing."""
    if M <= 256:
        o = (C.c_int * 2)()
        plan.few_rows(M, N, K, o)
        return {(o[0], o[1])}
    t = picked(plan, M, N, K)
    return {t[:2]} if t[2] > 1 else set()


def sliced_three(plan, M, qd, kd, d, K):
    o = (C.c_int * 2)()
    return {(o[0], o[1])} if plan.qkv(M, qd, kd, d, K, o) == 3 else set()


def gated(plan, M, F, K):
    return {((M + 31) // 32 * 32, plan.gated_columns(M, F, K))}


def test_gpu_tests_reach_every_sliced_tile(plan):
    """Whatever tile a cut can take, alone, over a pair or over K, Q and V, and whatever form gate and up of few rows
    can take, a GPU test launches."""
    one = set().union(*(sliced(plan, *s) for s in gpu.SPLIT_K))
    assert all(sliced(plan, *s) for s in gpu.SPLIT_K)
    few = set().union(*(sliced(plan, M, *nk) for M in gpu.FEW_ROWS for nk in gpu.FEW_ROWS_NK if not plan.direct(nk[0])))
    pair = set().union(*(sliced(plan, keep, (Hq + Hkv) * 128, D) for D, Hq, Hkv, keep in gpu.PAIRS))
    three, gate_up = set(), set()
    for M, D, Hq, Hkv, d, F in gpu.SIDE_BY_SIDE:
        three |= sliced_three(plan, M, Hq * d, Hkv * d, d, D)
        gate_up |= gated(plan, M, F, D) if M <= 256 else set()
    for M in list(range(257, 1025, 9)) + list(range(1025, 1537, 17)):
        for K in (256, 512, 768, 1024, 2048, 2304, 3584, 4096, 5120, 5888, 8192, 11008, 14336, 28672):
            for N in range(256, 12800, 256):
                assert sliced(plan, M, N, K) <= one, (M, N, K)
                if N % 512 == 0:
                    assert sliced(plan, M, N, K) <= pair, (M, N, K)
            for kd in (256, 384, 512, 640, 1024, 1408, 2048, 4096):
                for group in (1, 2, 4, 7, 8):
                    assert sliced_three(plan, M, kd * group, kd, 128, K) <= three, (M, kd * group, kd, K)
    for M in range(1, 257, 15):
        for K in (128, 256, 512, 768, 1024, 2048, 3584, 4096, 5120, 8192, 11008, 28672):
            for N in range(64, 16384, 320):
                assert plan.direct(N) or sliced(plan, M, N, K) <= few, (M, N, K)
            for F in range(128, 30000, 1280):
                assert gated(plan, M, F, K) <= gate_up, (M, F, K)
