"""The pool of page-locked staging buffers (csrc/pinned_pool.h), compiled against stand-ins
for the four runtime calls it makes: every allocation and every free happens in the
relaxed capture mode, the thread's own mode is restored after each, at most eight
buffers stay idle, and none is left once the last handle is gone."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "pinned_pool.h"
#include <stdio.h>
#include <stdlib.h>

static hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
static int g_live = 0, g_strict = 0, g_fail = 0, g_errors_read = 0;
extern "C" {
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    const hipStreamCaptureMode was = g_mode;
    g_mode = *m;
    *m = was;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    g_strict += g_mode != hipStreamCaptureModeRelaxed;
    if (g_fail) return hipErrorOutOfMemory;
    *p = malloc(n);
    ++g_live;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    g_strict += g_mode != hipStreamCaptureModeRelaxed;
    free(p);
    --g_live;
    return g_fail ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipGetLastError(void) { ++g_errors_read; return hipSuccess; }
}

#define CHECK(x) do { if (!(x)) { printf("line %d: %s (strict %d, live %d)\n", __LINE__, #x, g_strict, g_live); return 1; } } while (0)

int main()
{
    using namespace pcpic;
    PinnedPool pool;
    pool.add_handle();
    pool.add_handle();
    CHECK(pool.take(100, false).p == nullptr);
    PinnedPool::Block b[10];
    for (auto &k : b) k = pool.take(100, true);
    CHECK(g_live == 10 && b[0].n >= 100);
    for (auto &k : b) pool.give(k);
    CHECK(g_live == 8);                       // a ninth and a tenth idle buffer are given back
    const PinnedPool::Block large = pool.take(1 << 20, true);
    CHECK(large.n >= (1u << 20) && g_live == 9);
    pool.drop_handle();
    CHECK(g_live == 9);
    pool.drop_handle();                       // the last handle
    CHECK(g_live == 1);
    pool.give(large);                         // held past it
    CHECK(g_live == 0);
    CHECK(g_mode == hipStreamCaptureModeGlobal);
    CHECK(g_strict == 0);
    pool.add_handle();
    g_fail = 1;
    CHECK(pool.take(100, true).p == nullptr && g_errors_read == 1);
    g_fail = 0;
    pool.give(pool.take(100, true));
    g_fail = 1;
    pool.drop_handle();                       // an error of the free is not left for the next launch
    CHECK(g_errors_read == 2 && g_strict == 0 && g_mode == hipStreamCaptureModeGlobal);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pool_frees_in_relaxed_mode(tmp_path):
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_1011_6330_amd", "csrc"), str(src), "-o", str(exe), "-pthread"],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
