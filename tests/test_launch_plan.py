"""The rules of csrc/launch_plan.h, compiled on their own."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "launch_plan.h"
extern "C" {
void gather(int units, int G, long nblk, long n_static, int tau, int* got) {
  const mp::GatherPlan p = mp::plan_gather(units, G, nblk, n_static, tau);
  got[0] = p.run_blocks; got[1] = p.runs; got[2] = p.static_runs; got[3] = p.static_keys; got[4] = p.full;
}
long head_limit(int tuned, int G) { return mp::head_per_workgroup_limit(tuned, G); }
int hash_f32(int K, long groups32, long groups64) { return mp::hash_f32_keys(K, groups32, groups64); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    (tmp / "shim.cpp").write_text(SHIM)
    so = str(tmp / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2410_16179_amd", "csrc"), str(tmp / "shim.cpp"),
                    "-o", so], check=True)
    return ctypes.CDLL(so)


def gather(plan, units, G, n, n_static=68, tau=2):
    got = (ctypes.c_int * 5)()
    plan.gather(units, G, ctypes.c_long((n + 63) // 64), ctypes.c_long(n_static), tau, got)
    return tuple(got)


@pytest.mark.parametrize("units,G,n,n_static", [
    (64, 8, 1024, 1004), (64, 8, 2048, 68), (64, 8, 131072, 68), (8, 4, 16384, 4100), (8, 4, 16384, 16384), (1, 1, 64, 64), (64, 8, 65536, 6004),
    (80, 8, 10300, 700), (1, 4, 100000, 0), (512, 1, 4096, 516), (64, 8, 8192, 516), (260, 1, 200, 65)])
def test_gather_wavefronts_cover_the_blocks_and_share_the_static_set(plan, units, G, n, n_static):
    run_blocks, runs, own, keys, full = gather(plan, units, G, n, n_static)
    nblk = (n + 63) // 64
    assert run_blocks % 16 == 0 and run_blocks <= 128 and (runs - 1) * run_blocks < nblk <= runs * run_blocks
    assert full or run_blocks == 16                          # the form without full batches has a list for one piece
    # own wavefronts take the whole set; of keys dealt over the runs none gets more than two batches per piece, and no
    # more than half a batch where the runs leave the chip room
    if own:
        assert (own - 1) * keys < n_static <= own * keys and (full or keys == 32)
    else:
        share = -(-n_static // runs)
        assert share <= (64 * (run_blocks // 16) if units * runs * G >= 1024 else 16)
    # the partials fit the room that the workspace has for them
    assert runs + own <= -(-nblk // 16) + -(-n_static // 32)


def test_gather_forms_at_the_sizes_of_its_gpu_test(plan):
    # pieces of sixteen blocks per run, own static wavefronts and whether full batches have code of their own
    # (tests/test_gpu_gather_runs.py)
    def form(*a, **kw):
        run_blocks, _, own, keys, full = gather(plan, *a, **kw)
        return run_blocks // 16, (own, keys) if own else 0, bool(full)
    assert [form(64, 8, 10300), form(80, 5, 17000), form(128, 8, 35000)] == [(2, 0, True), (2, 0, True), (8, 0, True)]
    assert form(64, 8, 1000, 904) == (1, (15, 64), True)
    assert form(8, 4, 9000, 4131, tau=3) == (1, (65, 64), True)
    assert form(8, 4, 2500, 230, tau=3) == (1, (8, 32), False)
    assert form(8, 2, 3333, 3333, tau=3) == (1, (105, 32), False)
    assert form(260, 1, 200, 65) == (1, (3, 32), False)
    assert form(128, 8, 9000, 3000) == (3, (24, 128), True)
    assert form(8, 4, 16384, 68, tau=3) == (1, 0, False)


@pytest.mark.parametrize("K,groups32,keys", [
    (1, 256, 32), (2, 512, 32), (2, 1000, 32), (3, 2550, 32), (4, 257, 32), (4, 8192, 32),   # narrow tables: 32 throughout
    (5, 1002, 64), (8, 256, 32), (8, 384, 64), (8, 642, 32), (8, 1536, 64), (9, 760, 32), (10, 320, 64), (10, 515, 32), (10, 770, 64),
    (10, 2560, 64), (16, 258, 64), (16, 750, 32)])
def test_keys_of_a_float32_hashing_workgroup(plan, K, groups32, keys):
    # the faster of the two forms where they differ by more than a tenth; either where they do not
    assert plan.hash_f32(K, ctypes.c_long(groups32), ctypes.c_long((groups32 + 1) // 2)) == keys


@pytest.mark.parametrize("units,G,n,tuned,one", [
    # the sizes of tests/test_gpu_head_per_workgroup.py (up to 780 workgroups a run is four key blocks)
    (1, 4, 70, True, True), (8, 2, 1001, True, True), (8, 4, 2048, True, True), (8, 3, 1300, True, True), (2, 8, 4096, True, True), (4, 5, 777, True, True),
    (1, 7, 1500, False, True), (4, 3, 515, False, True), (8, 5, 1600, False, True), (8, 4, 6144, True, True), (8, 4, 6209, True, False), (1, 2, 3, True, True),
    # and those on which the limits rest
    (8, 2, 4096, True, True), (8, 2, 8192, True, False), (8, 2, 8192, False, False), (8, 3, 10000, True, False), (8, 4, 10000, True, False),
    (8, 4, 4096, False, True), (8, 4, 6144, False, False), (8, 5, 6400, True, True), (4, 7, 9000, True, True), (8, 8, 4000, False, True), (8, 8, 8000, True, False)])
def test_head_per_workgroup(plan, units, G, n, tuned, one):
    plan.head_limit.restype = ctypes.c_long
    assert (units * (-(-n // 256)) * G <= plan.head_limit(int(tuned), G)) == one
