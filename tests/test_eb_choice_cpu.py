"""The rule that chooses the kernel of a checked EmbeddingBag call (csrc/eb_choice.h, host code only), built here on its own."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_00130_amd", "csrc")
BATCH, GROUP1, GROUP2, GROUP4 = 0, 1, 2, 4
MOST = 2 ** 32 - 1      # work-items of one launch


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rule") / "rule.so")
    src = ('#include "eb_choice.h"\nextern "C" int pick(long long n, long long i, int p) { return abft::eb_pick_kernel(n, i, p); }\n'
           'extern "C" long long items(int k, long long n, int p) { return abft::eb_work_items((abft::EbKernel)k, n, p); }\n'
           'extern "C" int passes_by(long long stride, long long rows) { return abft::eb_passes_by(stride, rows); }\n')
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", "-x", "c++", "-", "-o", lib],
                   input=src, text=True, check=True)
    so = ctypes.CDLL(lib)
    so.pick.argtypes, so.items.argtypes, so.items.restype = [ctypes.c_longlong] * 2 + [ctypes.c_int], [ctypes.c_int, ctypes.c_longlong, ctypes.c_int], ctypes.c_longlong
    so.passes_by.argtypes = [ctypes.c_longlong] * 2
    return so


@pytest.mark.parametrize("pieces", [1, 2, 4, 8, 16, 32])
def test_no_launch_is_too_large(rule, pieces):
    """Whatever the batch kernel can run is run: never a kernel whose launch would have 2^32 work-items or more."""
    for n in [1, 999, 16000] + [2 ** e + o for e in range(20, 31) for o in (-1, 0, 1)]:
        for mean in (0, 1, 5, 6, 10, 11, 12, 16, 20, 30, 45, 46, 100, 1000):
            chosen = rule.pick(n, n * mean, pieces)
            assert chosen in (BATCH, GROUP1, GROUP2, GROUP4)
            if rule.items(BATCH, n, pieces) <= MOST:
                assert rule.items(chosen, n, pieces) <= MOST, (n, mean)


# (rows of 16, 32, 64, 128 and 512 bytes where a few lanes per lookup measured faster than a wavefront, and where they did not)
@pytest.mark.parametrize("pieces,n,mean,batch", [(1, 49152, 13, True), (1, 49152, 16, False), (1, 196608, 16, True), (1, 196608, 20, False), (2, 32768, 16, True),
                                                 (2, 32768, 25, False), (4, 80000, 20, True), (4, 98304, 12, True), (4, 98304, 25, False), (4, 16384, 12, False),
                                                 (8, 262144, 16, True), (8, 65536, 20, False), (16, 16384, 13, False), (32, 16384, 12, True),
                                                 (32, 16384, 16, False), (32, 65536, 20, True), (32, 65536, 32, False)])
def test_large_batches_of_longer_lookups(rule, pieces, n, mean, batch):
    assert (rule.pick(n, n * mean, pieces) == BATCH) == batch


@pytest.mark.parametrize("pieces,n,mean,kernel", [(4, 999, 60, GROUP4), (4, 1000, 60, GROUP2), (16, 1024, 30, GROUP4), (16, 1025, 30, GROUP1), (16, 1100, 60, GROUP2),
                                                  (32, 3999, 60, GROUP4), (32, 4000, 60, GROUP2), (32, 9999, 110, GROUP4), (32, 10000, 110, GROUP2), (32, 1100, 30, GROUP2), (8, 1279, 60, GROUP4),
                                                  (8, 1280, 60, GROUP2), (8, 1024, 110, GROUP4), (8, 1025, 110, GROUP2), (8, 1000, 30, GROUP1)])
def test_four_wavefronts_for_long_lookups_of_wide_rows(rule, pieces, n, mean, kernel):
    assert rule.pick(n, n * mean, pieces) == kernel


@pytest.mark.parametrize("stride,rows,by", [(80, 4_000_000, False), (80, 16_000_000, False), (80, 32_000_000, True), (272, 2_000_000, False), (272, 8_000_000, True),
                                            (528, 2 ** 40, True), (32, 1, False)])
def test_records_of_large_tables_pass_the_caches_by(rule, stride, rows, by):
    assert bool(rule.passes_by(stride, rows)) == by
