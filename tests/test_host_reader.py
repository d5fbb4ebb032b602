"""The reader of large device buffers (csrc/host_reader.h) on the CPU: compiled against a model of the few runtime calls it makes, in which work
given to the null stream is done when something waits for that stream, and streams belong to a device."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1509_03371_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <functional>
enum hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
enum { hipMemcpyDeviceToHost = 2, hipHostMallocDefault = 0, hipStreamNonBlocking = 1 };
typedef struct Stream { int unused; } *hipStream_t;
inline std::function<void()> null_stream;               // what was given to it and is not done
inline void drain() { if (null_stream) { auto f = std::move(null_stream); null_stream = nullptr; f(); } }
inline thread_local int current_device = 0;
inline std::atomic<bool> wrong_device{false};           // a stream was waited for or copied on from another device than its own
inline hipError_t hipGetDevice(int *d) { *d = current_device; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { current_device = d; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
inline hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = new Stream; return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t s) { if (current_device != 1) wrong_device = true; if (!s) drain(); return hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int, hipStream_t) { if (current_device != 1) wrong_device = true; memcpy(d, s, n); return hipSuccess; }
inline hipError_t hipMemcpy(void *d, const void *s, size_t n, int) { drain(); memcpy(d, s, n); return hipSuccess; }
"""

PROGRAM = r"""
#include <cstdio>
#include <new>
#include <vector>
#include "host_reader.h"
static thread_local int failing_new = 0;                // the failing_new-th allocation of this thread from now on finds no memory
void *operator new(size_t n)
{
    if (failing_new > 0 && --failing_new == 0) throw std::bad_alloc();
    void *p = malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
int main(int argc, char **argv)
{
    const size_t bytes = (argc > 1 ? atol(argv[1]) : 0);
    std::vector<unsigned char> src(bytes, 1), dst(bytes, 0);
    sk::HostReader reader;
    current_device = 1;                                 // the plan's device
    reader.open();
    current_device = 0;                                 // ... is not the caller's when it reads
    int made_on = -1;
    null_stream = [&] { for (size_t i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 7 + (i >> 20)); };
    const bool made = argc > 2 && argv[2][0] == 'm';                         // by a kernel, which must run on the plan's device
    if (argc > 2 && !made) failing_new = atoi(argv[2]);
    const hipError_t e = made ? reader.read_made(dst.data(), src.data(), bytes, [&](hipStream_t s) { made_on = s ? -2 : current_device; return hipSuccess; })
                              : reader.read(dst.data(), src.data(), bytes);
    failing_new = 0;
    if (current_device != 0 || (made && made_on != 1) || wrong_device) return 2;
    size_t wrong = e == hipSuccess ? 0 : bytes;
    for (size_t i = 0; i < bytes; ++i) wrong += dst[i] != (unsigned char)(i * 7 + (i >> 20));
    reader.close();
    printf("%zu\n", wrong);
    return wrong ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_reader")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(PROGRAM)
    exe = d / "reader"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(d), "-I", CSRC, "-o", str(exe), str(d / "main.cpp")], check=True)
    return str(exe)


# one piece, a piece and a byte, fewer pieces than lanes, many and a rest
@pytest.mark.parametrize("size", [1000, 2 << 20, (2 << 20) + 1, 5 << 20, (37 << 20) + 12345])
def test_reads_behind_the_null_stream(program, size):
    r = subprocess.run([program, str(size)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)


@pytest.mark.parametrize("size", [1000, (7 << 20) + 3])
def test_makes_and_reads_on_the_device_of_the_plan(program, size):
    r = subprocess.run([program, str(size), "made"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)


# the first, second and third thread's allocation fails: with none, one and two helpers running
@pytest.mark.parametrize("failing", [1, 2, 3])
def test_reads_all_without_memory_for_threads(program, failing):
    r = subprocess.run([program, str((23 << 20) + 3), str(failing)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
