"""conv_circular_noalloc allocates no host memory, also when no other convolution has run
in the process: a child process whose `operator new` is counted, by the library's own
calls of it, builds the plan with ntt_forward and then makes the call."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1005_1497_amd", "libnttmi.so")

COUNTER = r"""
#include <cstdlib>
#include <new>
static char *lo, *hi;
static long count;
extern "C" void watch(char* a, char* b) { lo = a; hi = b; count = 0; }
extern "C" long counted() { return count; }
static void* take(std::size_t n, void* caller) {
    if ((char*)caller >= lo && (char*)caller < hi) ++count;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(std::size_t n) { return take(n, __builtin_return_address(0)); }
void* operator new[](std::size_t n) { return take(n, __builtin_return_address(0)); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
void operator delete[](void* p, std::size_t) noexcept { std::free(p); }
"""

CHILD = r"""
import ctypes, sys
C = ctypes
counter = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)     # before anything that brings its own operator new
counter.watch.argtypes = [C.c_void_p, C.c_void_p]
counter.counted.restype = C.c_long
L = C.CDLL(sys.argv[2])
span = [l.split()[0].split("-") for l in open("/proc/self/maps") if l.rstrip().endswith("libnttmi.so")]
lo, hi = min(int(a, 16) for a, _ in span), max(int(b, 16) for _, b in span)
M = 13631489
order = C.c_uint32()
counter.watch(lo, hi)
assert L.ntt_modulus_order(C.c_uint64(M), C.byref(order)) == 0 and order.value == 19
assert counter.counted() > 0, "the library's allocations are not seen"
if sys.argv[3] == "cpu":
    sys.exit(0)
hip = C.CDLL("libamdhip64.so")
x = [C.c_void_p() for _ in range(3)]
for p in x:
    assert hip.hipMalloc(C.byref(p), C.c_size_t(4 << 19)) == 0
    assert hip.hipMemset(p, 0, C.c_size_t(4 << 19)) == 0
sig = [C.c_uint64, C.c_uint32, C.c_uint64, C.c_uint32]
L.ntt_forward.argtypes = sig + [C.c_void_p, C.c_void_p, C.c_uint32, C.c_uint32, C.c_void_p]
L.conv_circular_noalloc.argtypes = sig + [C.c_void_p] * 3 + [C.c_uint32, C.c_void_p]
for n in (8, 10, 13, 16, 19):
    root = pow(2, 1 << (19 - n), M)
    assert L.ntt_forward(M, n, root, 32, x[0], x[2], 1, 0, None) == 0
    counter.watch(lo, hi)
    assert L.conv_circular_noalloc(M, n, root, 32, x[0], x[1], x[2], 0, None) == 0
    took = counter.counted()
    assert hip.hipDeviceSynchronize() == 0
    print(n, took, flush=True)
    assert took == 0, (n, took)
"""


def run(tmp_path, where):
    src, lib, child = tmp_path / "counter.cpp", tmp_path / "libcounter.so", tmp_path / "child.py"
    src.write_text(COUNTER)
    child.write_text(CHILD)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    r = subprocess.run([sys.executable, str(child), str(lib), LIB, where], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_counter_sees_the_library(tmp_path):
    run(tmp_path, "cpu")


@pytest.mark.gpu
def test_noalloc_without_another_convolution(tmp_path):
    run(tmp_path, "gpu")
