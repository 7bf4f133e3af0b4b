"""Host check of the kept device scratch (csrc/scratch.cpp, compiled here
against a stand-in for the allocator with a limit): what is kept is bounded, is
given back when a volume ends and on demand, and never stands in the way of an
allocation of the library."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "scratch.cpp"
#include <map>
static std::map<void*, size_t> g_live;
static size_t g_limit = 0, g_used = 0;
static hipError_t g_last = hipSuccess;
static uintptr_t g_next = 4096;
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipMalloc(void** p, size_t n)
{
    if (g_used + n > g_limit) return g_last = hipErrorOutOfMemory;
    *p = (void*)g_next;
    g_next += (n + 4095) / 4096 * 4096;
    g_live[*p] = n;
    g_used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    auto it = g_live.find(p);
    if (it == g_live.end()) return hipErrorInvalidValue;
    g_used -= it->second;
    g_live.erase(it);
    return hipSuccess;
}
static sc::Scratch g_held[4];
extern "C" {
void limit(size_t n) { g_limit = n; }
size_t used() { return g_used; }
int last() { return (int)g_last; }
int take(int k, size_t n) { g_held[k] = sc::scratch_take(n); return g_held[k].p != nullptr; }
void give(int k, int idle) { sc::scratch_give(g_held[k], idle != 0); }
void volumes(int d) { sc::scratch_volumes(d); }
int alloc(size_t n) { void* p; return sc::device_alloc(&p, n); }
}
"""
MIB = 1 << 20


@pytest.fixture
def store(tmp_path):
    src, so = tmp_path / "store.cpp", tmp_path / "libstore.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}",
                           f"-I{os.path.join(ROOT, 'paper_1709_03763_amd', 'csrc')}", str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    L.used.restype = ctypes.c_size_t
    L.limit.argtypes = L.alloc.argtypes = [ctypes.c_size_t]
    L.take.argtypes = [ctypes.c_int, ctypes.c_size_t]
    L.limit(4096 * MIB)
    return L


def test_little_is_kept_without_a_volume(store):
    for size in (90, 300):
        assert store.take(0, size * MIB)
        store.give(0, 1)
        assert store.used() <= 128 * MIB
    assert store.used() >= 90 * MIB
    store.sc_release_scratch()
    assert store.used() == 0
    store.volumes(1)
    store.volumes(1)
    assert store.take(0, 100 * MIB)
    store.give(0, 1)
    kept = store.used()
    assert 100 * MIB <= kept <= 125 * MIB
    assert store.take(0, 99 * MIB)  # the kept one
    assert store.used() == kept
    store.volumes(-1)  # frees what is kept, not what is in use
    assert store.used() == kept
    store.give(0, 1)
    assert store.used() == kept
    store.volumes(-1)
    assert store.used() == 0


def test_kept_scratch_is_bounded(store):
    store.volumes(1)
    for k in range(4):
        assert store.take(k, 400 * MIB)
    for k in range(4):
        store.give(k, 1)
    assert store.used() <= 1024 * MIB
    assert store.take(0, 2000 * MIB)
    store.give(0, 1)
    assert store.used() <= 1024 * MIB
    assert store.take(0, 300 * MIB)
    store.give(0, 0)  # still in use by the device: freed, which waits
    store.volumes(-1)
    assert store.used() == 0


def test_kept_scratch_gives_way(store):
    store.volumes(1)
    assert store.take(0, 800 * MIB)
    store.give(0, 1)
    kept = store.used()
    assert kept >= 800 * MIB
    store.limit(1000 * MIB)
    assert store.alloc(900 * MIB)
    assert store.used() == 900 * MIB and store.last() == 0
    assert not store.take(0, 200 * MIB)  # no memory at all: refused, and no error left behind
    assert not store.alloc(200 * MIB)
    assert store.last() == 0
