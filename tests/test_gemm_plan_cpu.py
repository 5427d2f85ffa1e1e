"""The rules by which a checked product is laid out in its workspace (csrc/abft_internal.h, host code), built here on their own."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_00130_amd", "csrc")
SRC = """
#include "abft_internal.h"
extern "C" void plan(int M, int N, int K, int stages, int whole, long long* out) {
    const abft::SplitKPlan s = abft::splitk_plan(M, N, stages, whole != 0);
    const abft::RealignPlan r = abft::realign_plan(M, N, K, stages);
    const abft::Split64Plan l = abft::split64_plan(M, N, stages);
    const long long v[] = {s.z, (long long)s.tickets_off, (long long)s.part_off, (long long)s.total_ints, (long long)s.room_ints, r.copy, (long long)r.off,
                           (long long)r.total_ints, (long long)abft::ws_base_ints(M), l.z, (long long)l.total_ints};
    for (int i = 0; i < 11; ++i) out[i] = v[i];
}
extern "C" int form(int M, int N, int stages, int whole) { return abft::wk_form(M, N, stages, whole != 0); }
extern "C" int room_for_copy(int M, int N, int K) { return abft::room_for_copy(M, N, K); }
extern "C" int beyond(int M, int N, int stages) { return abft::beyond_wk_form(M, N, stages); }
extern "C" int large(int M, int N, int K, int stages, int whole, int can_copy, int pick, int pick_copy, int want_c, int want_q, int check) {
    const abft::LargeChoice c = abft::large_choice({(abft::LargeForm)pick, pick_copy != 0}, whole != 0, can_copy != 0, M, N, K, stages, want_c != 0, want_q != 0, check != 0);
    return c.form + (c.copy ? 8 : 0);
}
extern "C" void packed(int K, int N, long long* out) {
    const int KB = (K + 127) / 128 * 2, NT = (N + 255) / 256;
    const abft::PackedLayout l = abft::packed_layout(KB, NT);
    const long long v[] = {(long long)NT * 256 * KB * 64, 0, (long long)l.limbs, (long long)l.limbs127, (long long)l.S_B, (long long)l.colsum, (long long)l.total, (long long)l.S_B127,
                           (long long)l.sums, (long long)l.bytes, KB * 64, NT * 256};
    for (int i = 0; i < 12; ++i) out[i] = v[i];
}
extern "C" int slots(int M, int tiles_n) { return abft::row_slots(M, tiles_n).slots; }
extern "C" int slot_rows(int M, int tiles_n) { return abft::row_slots(M, tiles_n).rows; }
extern "C" int copy_first(int form, int stages) { return abft::copy_first((abft::WkForm)form, stages); }
"""
NONE, T32X32W4, T32X32W8, T32X64W4, T32X64W8, T64X64W4 = range(6)


class Plan:
    def __init__(self, v):
        self.z, self.tickets_off, self.part_off, self.split_ints, self.room_ints, self.copy, self.copy_off, self.copy_ints, self.words, self.z64, self.split64_ints = v


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "plan.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-shared", "-fPIC", f"-I{CSRC}", f"-I{rocm}/include", "-x", "c++", "-",
                    "-o", lib], input=SRC, text=True, check=True)
    so = ctypes.CDLL(lib)

    def call(M, N, K, whole):
        out = (ctypes.c_longlong * 11)()
        so.plan(M, N, K, ((K + 63) // 64 + 1) // 2, whole, out)
        return Plan(out)
    call.room_for_copy = lambda M, N, K: bool(so.room_for_copy(M, N, K))
    call.copy_first = lambda form, K: bool(so.copy_first(form, ((K + 63) // 64 + 1) // 2))
    call.form = lambda M, N, K: so.form(M, N, ((K + 63) // 64 + 1) // 2, K % 16 == 0)
    call.packed = lambda K, N: (lambda out: (so.packed(K, N, out), list(out))[1])((ctypes.c_longlong * 12)())
    call.slots = lambda M, tiles_n: (so.slots(M, tiles_n), so.slot_rows(M, tiles_n))
    call.beyond = lambda M, N, K: bool(so.beyond(M, N, ((K + 63) // 64 + 1) // 2))
    call.large = lambda M, N, K, pick, out="C", can_copy=False, check=True: so.large(M, N, K, ((K + 63) // 64 + 1) // 2, K % 16 == 0, can_copy, pick & 7, pick >> 3,
                                                                         out != "q", out != "C", check)
    return call


SIZES = [1, 16, 32, 33, 40, 41, 48, 64, 65, 128, 129, 200, 256, 500, 512, 1000, 4097]
WIDTHS = [1, 32, 33, 64, 100, 200, 256, 500, 1000, 1500, 4096, 4200, 6500, 9000]
DEPTHS = [17, 385, 2049, 2999, 3071, 3073, 4609, 5001, 6145, 8191, 9001, 16383, 40001]


def test_copy_and_parts_lie_apart(plan):
    """Wherever a call may both copy the rows of A and split K (its copy has whole rows), neither area reaches into the other, nor
    into the words, and a workspace that holds the copy holds the parts too."""
    both = both64 = 0
    for M in SIZES:
        for N in WIDTHS:
            for K in DEPTHS:
                p = plan(M, N, K, 1)
                assert p.words <= p.tickets_off < p.part_off
                if p.copy:
                    assert p.copy_off >= p.part_off and p.copy_ints >= p.copy_off + M * ((K + 15) // 16 * 16) // 4
                if p.copy and p.z > 1:
                    both += 1
                    assert p.copy_off >= p.split_ints, (M, N, K, p.z)
                if p.copy and p.z64 > 1:
                    both64 += 1
                    assert p.copy_off >= p.split64_ints, (M, N, K, p.z64)
                for whole in (0, 1):
                    s = plan(M, N, K, whole)
                    assert s.z == 1 or s.split_ints <= s.room_ints, (M, N, K)
    assert both > 50 and both64 > 5


# (shapes where the streaming kernel measured faster for weights that have not just been used, and neighbours where it did not)
@pytest.mark.parametrize("M,N,K,streams", [(1, 800, 2048, True), (1, 800, 3200, True), (4, 4096, 4096, True), (8, 2048, 4096, True), (1, 3000, 12000, True), (8, 3000, 16384, False), (8, 3500, 12000, True), (4, 2500, 12000, False), (4, 774, 5280, True),
                                           (8, 12000, 1024, True), (1, 15000, 3008, True), (16, 4096, 2048, True), (10, 464, 4064, True), (1, 800, 2560, False), (1, 832, 5312, True), (2, 832, 5312, True), (2, 1200, 5312, False), (1, 832, 4400, False),
                                           (8, 3000, 6400, False), (8, 800, 6400, False), (16, 4096, 4096, False), (16, 1200, 2048, False), (4, 12000, 1152, False),
                                           (8, 15000, 3008, True), (8, 15000, 5008, False), (4, 15000, 5008, True), (8, 8192, 1001, True), (1, 4096, 9001, True), (3, 3000, 9008, False), (1, 16384, 3008, False), (24, 800, 2048, False), (8, 4096, 512, False), (1, 800, 3201, True),
                                           (1, 300, 2001, True), (1, 800, 1001, True), (4, 300, 2001, True), (1, 6001, 9001, True), (4, 800, 3201, False), (8, 3000, 2049, False),
                                           (1, 800, 500, False), (1, 8192, 16383, False), (2, 800, 1001, False), (16, 300, 2001, False)])
def test_few_rows(plan, M, N, K, streams):
    assert (plan.form(M, N, K) == NONE) == streams


# (one or two stages of many rows, where the 64x64 tiles measured faster, and neighbours where they did not)
@pytest.mark.parametrize("M,N,K,form", [(3000, 64, 128, NONE), (2739, 80, 112, NONE), (3000, 128, 256, NONE), (1056, 300, 128, NONE), (1500, 64, 112, NONE),
                                        (1500, 128, 112, T32X32W4), (2100, 100, 256, T32X64W4), (1056, 64, 256, T32X32W4), (3000, 32, 112, T32X32W4),
                                        (3000, 128, 384, T32X64W4), (2739, 80, 115, T32X64W4), (1000, 64, 128, T32X32W4)])
def test_many_rows_of_a_short_k(plan, M, N, K, form):
    assert plan.form(M, N, K) == form


# (rows that are no whole chunks: a copy first for the 64x64 form and a long K, with a workspace that has the room)
@pytest.mark.parametrize("M,N,K,copied", [(64, 12000, 5001, True), (128, 6500, 9001, True), (256, 3000, 5001, True), (100, 5000, 2001, False), (64, 5000, 9001, False),
                                          (33, 8192, 9001, False), (2000, 1000, 479, False)])
def test_copy_ahead_of_the_large_form(plan, M, N, K, copied):
    form = plan.form(M, N, K)
    assert form != NONE and plan.copy_first(form, K) == copied
    if copied:      # the copy is one that is made, the whole rows then run on 64x64 tiles of the same kernel, and M > 32 leaves room for it
        assert plan(M, N, K, 0).copy and plan.form(M, N, (K + 15) // 16 * 16) == T64X64W4 and M > 32


# (where the 64x64 tiles with a split K measured faster, by slices, and neighbours where they did not)
@pytest.mark.parametrize("M,N,K,z", [(64, 4200, 9008, 3), (64, 5000, 16000, 3), (33, 5000, 9008, 3), (64, 3000, 12000, 5), (64, 2000, 16000, 8), (64, 6500, 16000, 2),
                                     (40, 1360, 20496, 11), (64, 5000, 6000, 1), (33, 3000, 12000, 1), (64, 2000, 9008, 1), (64, 6500, 9008, 1), (64, 1000, 16000, 1),
                                     (164, 1440, 15312, 3), (746, 339, 14848, 3), (192, 1500, 9008, 1), (130, 1400, 11600, 1), (1100, 250, 12000, 3), (128, 3000, 12000, 1), (128, 1500, 16000, 1), (65, 4200, 9008, 1), (32, 4200, 9008, 1), (64, 9000, 16000, 1)])
def test_split_of_the_large_tiles(plan, M, N, K, z):
    p = plan(M, N, K, 1)
    assert p.z64 == z
    if z > 1:
        tiles = (M + 63) // 64 * ((N + 63) // 64)
        assert 128 < tiles * z <= 256 and tiles <= p.part_off - p.tickets_off and p.split64_ints == p.part_off + tiles * z * (256 * 17 + 64)


def test_calls_of_rows_that_are_no_whole_chunks(plan):
    """Wherever the library copies such rows on its own account the workspace has room for the copy; and of up to 32 rows only calls that the
    streaming kernel takes at any alignment are left to it (up to 16 rows, or more than 8192 columns)."""
    copies = left = 0
    for M in [*range(1, 34), 40, 41, 48, 49, 64, 65, 100, 128, 200, 256, 500, 1000, 3000, 9000]:
        for N in (1, 40, 300, 900, 1345, 2000, 3000, 4096, 4097, 4161, 6500, 8191, 8193, 12000, 16383, 16384, 16385, 20000, 33000, 70000):
            for K in (17, 129, 500, 1001, 1999, 2999, 4095, 4097, 6001, 9001, 12001, 15361, 16383, 33001):
                form = plan.form(M, N, K)
                if M <= 32 and form == NONE:
                    left += 1
                    assert M <= 16 or N > 8192, (M, N, K)
                p = plan(M, N, K, 0)
                if M > 32 and p.copy and (form == NONE or plan.copy_first(form, K) or p.z64 > 1):
                    copies += 1
                    assert plan.room_for_copy(M, N, K), (M, N, K)
    assert copies > 100 and left > 100


# (slices of 32x32 tiles with rows of whole chunks; where two or three pay, and neighbours that run unsplit)
@pytest.mark.parametrize("M,N,K,z", [(64, 64, 16384, 8), (46, 128, 13504, 7), (32, 3000, 12000, 2), (16, 2500, 9008, 3), (64, 1100, 12000, 3), (64, 1500, 9008, 2),
                                     (256, 500, 12000, 2), (1280, 80, 16176, 2), (100, 1000, 12000, 1), (33, 2000, 12000, 1), (128, 1000, 8192, 1), (32, 3000, 8192, 1)])
def test_split_of_the_small_tiles(plan, M, N, K, z):
    p = plan(M, N, K, 1)
    assert p.z == z and (z == 1 or (p.split_ints <= p.room_ints and 4 * ((M + 31) // 32) * ((N + 31) // 32) <= p.part_off - p.tickets_off))


def test_grids_beyond_the_compute_units(plan):
    """What the fits choose there: small tiles for a short K and for grids that large ones would leave idle, large ones for many rows, columns
    and a long K; a copy only where there is room for one; never where wk_form has a rule."""
    L256, L128, L64, W32X64, W64X64, COPY = 0, 1, 2, 3, 4, 8
    assert plan.large(2545, 7104, 528, L256, "both") == L64 and plan.large(3350, 2688, 288, L256, "both") == L64
    assert plan.large(4096, 4096, 4096, L256) == L256 and plan.large(4096, 4096, 1024, L256, "q") == L256 and plan.large(2048, 2048, 4096, L128) == L128
    assert plan.large(90, 8237, 3824, L64, "q") == W32X64 and plan.large(214, 4369, 2434, L64 + COPY, "both", True) == W32X64
    assert plan.large(2085, 506, 12288, L64) in (W32X64, W64X64)
    for M in (33, 64, 100, 300, 1000, 4096, 100000):
        for N in (100, 1000, 4000, 16384):
            for K in (17, 64, 100, 500, 1040, 4096, 9001):
                if not plan.beyond(M, N, K):
                    continue
                assert plan.form(M, N, K) in (NONE, T32X64W4, T64X64W4)
                for out in ("C", "q", "both"):
                    for pick in (L256, L128, L64):
                        assert plan.large(M, N, K, pick, out) < COPY
                        assert plan.large(M, N, K, pick + (COPY if K % 16 else 0), out, True) in ((L256, L128, L64, W32X64, W64X64) if K % 16 == 0 else
                                                                                                 (L64, W32X64, W64X64, *(COPY + f for f in range(5))))
    assert plan.beyond(131072, 258, 32) and not plan.beyond(131073, 258, 32)    # (row words that reach into the scratch)
    assert not plan.beyond(32, 100000, 4096) and not plan.beyond(64, 256, 512) and not plan.beyond(1024, 1024, 4096) and plan.beyond(1024, 1040, 4096)


def test_grids_beyond_the_compute_units_where_the_fits_are_off(plan):
    """A few tiles more than two to each compute unit and a long K, outputs beyond the memory-side cache, gains within the fits' error: what the
    thresholds choose stays."""
    L256, L128, L64, W32X64, W64X64 = 0, 1, 2, 3, 4
    for M, N, K in ((524, 3629, 9632), (389, 4800, 7312), (174, 10928, 5344)):    # 513 to 525 tiles of 64x64
        assert plan.large(M, N, K, L128) == L128
    assert plan.large(304, 6180, 6224, L128) == W64X64 and plan.large(776, 4703, 4368, L128, "both") == W64X64    # 485, 962
    for M, N in ((16400, 8240), (8200, 16480), (32800, 4120), (43102, 2096), (20853, 3600)):    # 286 to 515 MiB
        assert plan.large(M, N, 96, L256) == L256
    assert plan.large(16400, 2060, 96, L256) == L64 and plan.large(8200, 4120, 96, L256) == L64    # 129
    assert plan.large(2824, 15456, 112, L256) == L256 and plan.large(555, 115760, 96, L256) == L256    # 167 and 245, long rows
    assert plan.large(1238, 15574, 160, L256) == L64 and plan.large(2472, 13264, 96, L256, "both") == L64    # 74, and both outputs
    # predicted 0.91 to 0.94 of the thresholds' choice; 0.88, unchecked as well
    assert plan.large(297, 7168, 3056, L128, "q") == L128 and plan.large(1295, 14192, 2256, L256, "q") == L256 and plan.large(314, 111907, 1616, L256) == L256
    assert plan.large(414, 1607, 336, L64) == W32X64 and plan.large(414, 1607, 336, L64, check=False) == L64


@pytest.mark.parametrize("K,N", [(1, 1), (64, 256), (129, 257), (300, 16384), (16385, 20), (1024, 1024), (4096, 4096), (16384, 16384)])
def test_what_a_packed_weight_takes(plan, K, N):
    """Digits, sums and totals beside the weight itself: 20 bytes a row and 8 a column of it (accumulators among them), whatever the number of tiles."""
    units, *at, total, k, n = plan.packed(K, N)
    ints = (k, k, k, n, 64, k)    # 4 bytes a place: both kinds of digits, S_B, colsum, the totals, S_B mod 127
    assert at[0] == 0 and at[1] == units
    for i, count in enumerate(ints):
        assert at[i + 1] % 256 == 0 and at[i + 2] - at[i + 1] >= 4 * count
    assert total == at[-1] + 4 * (k + n) and total - units <= 24 * k + 8 * n + 8 * 256
    if K >= 4096 and N >= 4096:
        assert total <= 1.01 * units


def test_slots_of_the_row_words(plan):
    """Two kernels index the workspace by them: slots and the row words behind them lie within the words that every call has, a slot has a word
    for every row, and every slot meets at least one tile column (one that nobody arrives at would be waited for)."""
    words = (plan(1, 64, 64, 1).words - 64) // 2    # the least that a workspace holds
    for M in range(1, 400):
        for tiles_n in (1, 31, 32, 33, 48, 49, 50, 63, 64, 65, 150, 1000, 131072):
            n, rows = plan.slots(M, tiles_n)
            if tiles_n <= 48 or M > 384:
                assert (n, rows) == (0, 0)
                continue
            assert n >= 4 and n & (n - 1) == 0 and n < tiles_n and rows >= M
            assert (n + 1) * rows <= words and n == (32 if M <= 64 else 8 if M <= 192 else 4)
