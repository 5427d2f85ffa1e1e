"""Which blocks of destroyed weights are used again, and when the device is waited for (csrc/kept_blocks.h, host code), on a simulated device."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_00130_amd", "csrc")
SRC = """
#include <map>
#include "kept_blocks.h"
struct Device {                       // blocks are numbers from 1 on
    std::map<long, size_t> held;
    std::map<long, long> put_at;      // time of its last release by its weight
    long next = 1, now = 0, waited = -1, allocations = 0, releases = 0, waits = 0, early = 0;
    size_t bytes = 0, most = ~(size_t)0;
    int idle = 0, refuses = 0;
};
struct Memory {
    Device* d = nullptr;
    hipError_t allocate(void** out, size_t size) {
        if (d->bytes + size > d->most) return hipErrorOutOfMemory;
        d->held[d->next] = size;
        d->bytes += size;
        ++d->allocations;
        *out = (void*)d->next++;
        return hipSuccess;
    }
    bool release(void* p) {
        if (d->refuses) return false;
        d->bytes -= d->held.at((long)p);
        d->held.erase((long)p);
        ++d->releases;
        d->waited = d->now++;         // (hipFree waits for the device)
        return true;
    }
    bool wait() {
        if (d->refuses) return false;
        ++d->waits;
        d->waited = d->now++;
        return true;
    }
};
struct Sim {
    Device d;
    abft::KeptBlocks<Memory> kept{Memory{&d}};
};
extern "C" {
Sim* make() { return new Sim; }
void drop(Sim* s) { delete s; }
void set(Sim* s, int idle, size_t most, int refuses) { s->d.idle = idle; s->d.most = most; s->d.refuses = refuses; }
long get(Sim* s, size_t need, size_t* size) {
    void* p = nullptr;
    uint64_t mark = ~0ull;
    if (s->kept.get(need, &p, size, &mark, [s] { return s->d.idle != 0; }) != hipSuccess) return 0;
    const long b = (long)p;
    if (s->d.held.at(b) != *size || *size < need) return -1;
    if (mark != (s->d.put_at.count(b) ? 1000 + b : 0)) return -1;
    if (s->d.put_at.count(b) && s->d.put_at[b] > s->d.waited) ++s->d.early;    // handed out before a wait
    return b;
}
void put(Sim* s, long b, size_t size) {
    s->d.put_at[b] = s->d.now++;
    s->kept.put((void*)b, size, 1000 + b, true, [s] { return s->d.idle > 1; });
}
int trim(Sim* s) { return s->kept.trim(); }
void counts(Sim* s, long* out) {
    const long v[] = {s->d.allocations, s->d.releases, s->d.waits, s->d.early, (long)s->d.held.size(), (long)s->d.bytes};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}
}
"""
MIB = 1 << 20


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("kept") / "kept.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-shared", "-fPIC", f"-I{CSRC}", f"-I{rocm}/include", "-x", "c++", "-",
                    "-o", lib], input=SRC, text=True, check=True)
    so = ctypes.CDLL(lib)
    so.make.restype = ctypes.c_void_p
    so.drop.argtypes = [ctypes.c_void_p]
    so.set.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t, ctypes.c_int]
    so.get.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.POINTER(ctypes.c_size_t)]
    so.get.restype = ctypes.c_long
    so.put.argtypes = [ctypes.c_void_p, ctypes.c_long, ctypes.c_size_t]
    so.trim.argtypes = [ctypes.c_void_p]
    so.counts.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_long)]
    return so


class Sim:
    def __init__(self, so):
        self.so, self.at = so, so.make()

    def idle(self, idle, most=(1 << 64) - 1, refuses=0):
        self.so.set(self.at, idle, most, refuses)

    def pack(self, need):
        size = ctypes.c_size_t()
        b = self.so.get(self.at, need, ctypes.byref(size))
        assert b >= 0
        return (b, size.value) if b else None

    def destroy(self, weight):
        self.so.put(self.at, *weight)

    def replace(self, weight, need=None):
        new = self.pack(need or weight[1])
        self.destroy(weight)
        return new

    @property
    def n(self):
        v = (ctypes.c_long * 6)()
        self.so.counts(self.at, v)
        d = dict(zip(("allocations", "releases", "waits", "early", "held", "bytes"), v))
        assert d["early"] == 0, "a block was handed out that the device had not been waited for since its release"
        return d


@pytest.fixture
def sim(so):
    s = Sim(so)
    yield s
    so.drop(s.at)


def test_a_weight_replaced_again_and_again_waits_once_for_several(sim):
    """The same whatever the rate: nothing but the blocks counts."""
    w = sim.pack(16 * MIB)
    waits = []
    for i in range(200):
        before = sim.n["waits"]
        w = sim.replace(w)
        waits.append(sim.n["waits"] - before)
    assert max(waits) == 1 and sum(waits[20:]) <= 180 // 8 + 1
    assert not any(a and b for a, b in zip(waits, waits[1:]))
    assert sim.n["allocations"] == 9 and sim.n["releases"] == 0    # eight and the one in use, no more


def test_a_weight_replaced_on_an_idle_device_keeps_one_block(sim):
    sim.idle(1)
    w = sim.pack(16 * MIB)
    for i in range(50):
        w = sim.replace(w)
    n = sim.n
    assert n["allocations"] == 2 and n["held"] == 2 and n["waits"] == 49
    sim.idle(0)    # then a run of them
    n = sim.n
    for i in range(100):
        w = sim.replace(w)
    assert sim.n["allocations"] == 9 and sim.n["waits"] - n["waits"] <= 100 // 8 + 1


def test_a_weight_destroyed_on_an_idle_device_is_waited_for_at_once(sim):
    """... so that the next one, whose stream will be busy, finds a block; not again while there is one."""
    sim.idle(2)
    held = [sim.pack(16 * MIB) for _ in range(3)]
    sim.destroy(held.pop())
    assert sim.n["waits"] == 1
    sim.destroy(held.pop())
    assert sim.n["waits"] == 1
    sim.idle(0)
    held.append(sim.pack(16 * MIB))
    n = sim.n
    assert n["allocations"] == 3 and n["waits"] == 1
    sim.idle(2)
    sim.destroy(held.pop())
    assert sim.n["waits"] == 2


def test_large_blocks(sim):
    w = sim.pack(100 * MIB)    # two of them may be kept
    for i in range(30):
        w = sim.replace(w)
    assert sim.n["allocations"] == 3 and sim.n["waits"] == 14
    big = sim.pack(300 * MIB)
    big = sim.replace(big)
    assert sim.n["releases"] == 1    # more than is kept
    sim.destroy(w)
    sim.destroy(big)
    n = sim.n
    assert n["held"] == 0 and n["bytes"] == 0 and n["releases"] == n["allocations"]    # all given back with the last weight


def test_blocks_of_weights_that_are_gone_make_room(sim):
    """Sixteen weights of other sizes are destroyed; the one that goes on to be replaced gets blocks of its own size all the same."""
    other = [sim.pack((1 + i) * MIB * 2) for i in range(15)] + [sim.pack(300000)]    # 240 MiB
    w = sim.pack(7 * MIB + 4096)
    for b in other:
        sim.destroy(b)
    for i in range(48):    # (they are given back one by one once 32 releases lie behind theirs)
        w = sim.replace(w)
    before = sim.n
    for i in range(100):
        w = sim.replace(w)
    n = sim.n
    assert n["allocations"] - before["allocations"] <= 4 and n["releases"] - before["releases"] <= 4
    assert n["waits"] - before["waits"] <= 100 // 8 + 1


@pytest.mark.parametrize("weights", [2, 5, 10, 16, 24])
def test_weights_of_several_sizes_replaced_in_turn(sim, weights):
    w = [sim.pack((1 + i) * MIB // 2) for i in range(weights)]
    for i in range(10 * weights):
        w[i % weights] = sim.replace(w[i % weights])
    before = sim.n
    rounds = 50
    for i in range(rounds * weights):
        w[i % weights] = sim.replace(w[i % weights])
    n = sim.n
    # (more sizes than blocks are kept of: those that there is no room for are allocated and freed)
    assert n["allocations"] - before["allocations"] <= (rounds * weights // 10 if weights <= 16 else rounds * (weights - 16))
    assert n["waits"] - before["waits"] <= 2 * rounds and n["bytes"] - sum(b[1] for b in w) <= 256 * MIB


def test_sizes_that_come_once(sim):
    w = sim.pack(MIB)
    for i in range(200):
        sim.destroy(sim.pack((40 + 3 * i % 200) * MIB))
        n = sim.n
        assert n["held"] <= 17 and n["bytes"] <= 256 * MIB + w[1]


def test_a_wait_that_is_refused_makes_nothing_idle(sim):
    """As while another thread captures a graph: what has not been waited for is not handed out (Sim.n looks)."""
    w = sim.pack(100 * MIB)
    sim.idle(0, refuses=1)
    for i in range(10):
        w = sim.replace(w)
    assert sim.n["waits"] == 0 and sim.n["allocations"] == 11
    sim.idle(1)
    w = sim.replace(w)
    assert sim.n["waits"] == 1 and sim.n["allocations"] == 11


def test_what_cannot_be_given_back_is_kept(sim):
    """The last weight goes while hipFree is refused: its block and the kept ones serve later weights, or are given back with the last of those."""
    w = sim.pack(MIB)
    for i in range(5):
        w = sim.replace(w)
    sim.idle(0, refuses=1)
    sim.destroy(w)
    assert sim.n["held"] == 6 and sim.n["releases"] == 0
    sim.idle(1)
    sim.destroy(sim.pack(MIB))
    n = sim.n
    assert n["held"] == 0 and n["allocations"] == 6


def test_kept_blocks_are_given_back_when_asked_for(sim):
    w = sim.pack(MIB)
    for i in range(5):
        w = sim.replace(w)
    assert sim.so.trim(sim.at) and sim.n["held"] == 1
    w = sim.replace(w)
    sim.idle(0, refuses=1)
    assert not sim.so.trim(sim.at) and sim.n["held"] == 2
    sim.idle(0)
    assert sim.so.trim(sim.at) and sim.n["held"] == 1


def test_a_block_serves_weights_of_about_its_size(sim):
    sim.idle(1)
    held = sim.pack(MIB)
    sim.destroy(sim.pack(16 * MIB))
    small = sim.pack(14 * MIB)    # (an eighth of it would lie idle for as long as the weight lives)
    assert small[1] == 14 * MIB
    assert sim.pack(15 * MIB + MIB // 2)[1] == 16 * MIB
    assert held


def test_no_memory_for_a_new_block(sim):
    a, b = sim.pack(10 * MIB), sim.pack(50 * MIB)
    sim.destroy(a)
    sim.idle(0, 90 * MIB)
    c = sim.pack(40 * MIB)    # (the kept ten are given back)
    assert c and sim.n["held"] == 2
    assert sim.pack(40 * MIB) is None
    sim.destroy(b)
    assert sim.pack(40 * MIB)
