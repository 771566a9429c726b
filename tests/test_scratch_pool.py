"""Idle call scratch on the host: csrc/scratch.cpp compiled against a counted stand-in for the device allocator."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_14454_amd", "csrc")
HIPCC = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)),
             None)

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <map>
static std::map<void*, size_t> live;
static size_t used = 0, limit = size_t(1) << 40;
static int device = 0, mallocs = 0;
static hipError_t fake_malloc(void** p, size_t n) {
    ++mallocs;
    if (used + n > limit) return hipErrorOutOfMemory;
    static size_t next = 1 << 20;
    *p = reinterpret_cast<void*>(next);
    next += n;
    live[*p] = n;
    used += n;
    return hipSuccess;
}
static hipError_t fake_free(void* p) {
    if (!live.count(p)) std::printf("FAIL free of unknown pointer\n");
    used -= live[p];
    live.erase(p);
    return hipSuccess;
}
#define hipMalloc(p, n) fake_malloc(p, n)
#define hipFree(p) fake_free(p)
#define hipMemset(p, v, n) hipSuccess
#define hipGetDevice(d) (*(d) = device, hipSuccess)
#define hipGetLastError() hipSuccess
#include "scratch.cpp"
using namespace dwf;
#define CHECK(c) do { if (!(c)) std::printf("FAIL line %d: %s\n", __LINE__, #c); } while (0)
constexpr size_t GB = size_t(1) << 30;

int main() {
    {   // one shape: buffers go from call to call and from operator to operator; other shapes, classes, devices do not get them
        ScratchUser a, b;
        a.attach(8, 100);
        b.attach(8, 100);
        void *p, *q;
        { Scratch x({device, 0, 8, 100}, 64), y({device, 0, 8, 100}, 64); p = x.p; q = y.p; CHECK(p != q); }
        { Scratch x(a.key(0), 64), y(b.key(0), 64); CHECK(x.p != y.p && (x.p == p || x.p == q) && (y.p == p || y.p == q)); }
        CHECK(mallocs == 2 && used == 128);
        { Scratch x({device, 1, 8, 100}, 64); CHECK(x.p != p && x.p != q); }
        { Scratch x({device, 0, 7, 100}, 64); CHECK(x.p != p && x.p != q); }   // no such operator: freed again
        { Scratch x({device, 0, 8, 99}, 64); CHECK(x.p != p && x.p != q); }
        device = 1;
        ScratchUser d;
        d.attach(8, 100);
        { Scratch x({device, 0, 8, 100}, 64); CHECK(x.p != p && x.p != q); }
        device = 0;
        CHECK(used == 4 * 64);
        { ScratchUser c; c.attach(8, 100); }
        CHECK(used == 4 * 64);   // a and b are still there
        CHECK(release_scratch() && used == 0 && !release_scratch());
        { Scratch x({device, 0, 8, 100}, 64); }
        CHECK(used == 64);
    }
    CHECK(used == 0);   // the last operator of the shape is gone
    {   // a scope left by an exception frees its buffer
        ScratchUser a;
        a.attach(8, 100);
        try { Scratch x({device, 0, 8, 100}, 64); throw 1; } catch (int) {}
        CHECK(used == 0);
    }
    {   // the bound holds over all shapes, the oldest goes first, a buffer beyond it is not kept
        ScratchUser a, b, c;
        a.attach(2, 1);
        b.attach(3, 1);
        c.attach(4, 1);
        { Scratch x({device, 0, 2, 1}, 3 * GB); }
        { Scratch x({device, 0, 3, 1}, 3 * GB); }
        CHECK(used == 6 * GB);
        { Scratch x({device, 0, 4, 1}, 4 * GB); }
        CHECK(used == 7 * GB);
        const int n = mallocs;
        { Scratch x({device, 0, 3, 1}, 3 * GB); }
        CHECK(mallocs == n);
        { Scratch x({device, 0, 2, 1}, 3 * GB); }   // of 2: freed before
        CHECK(mallocs == n + 1 && used <= SCRATCH_IDLE_MAX);
        { Scratch x({device, 0, 2, 1}, SCRATCH_IDLE_MAX + 1); }
        CHECK(used <= SCRATCH_IDLE_MAX);
        { Scratch x({device, 0, 2, 1}, SCRATCH_IDLE_MAX); }
        CHECK(used == SCRATCH_IDLE_MAX);
        {
            Scratch x({device, 0, 2, 1}, SCRATCH_IDLE_MAX), y({device, 0, 3, 1}, 3 * GB);   // in use: not counted
            CHECK(used == SCRATCH_IDLE_MAX + 3 * GB);
        }
        CHECK(used <= SCRATCH_IDLE_MAX);
    }
    CHECK(used == 0);
    {   // no memory: idle buffers go, the allocation succeeds; without any it fails with its status
        ScratchUser a;
        a.attach(2, 1);
        { Scratch x({device, 0, 2, 1}, 2 * GB), y({device, 0, 2, 1}, 2 * GB); }
        CHECK(used == 4 * GB);
        limit = 5 * GB;
        { DevBuf b(3 * GB); CHECK(b.p && used == 3 * GB); }
        { Scratch x({device, 0, 2, 1}, 2 * GB); }
        int code = 0;
        try { DevBuf b(6 * GB); } catch (const Error& e) { code = e.code; }
        CHECK(code == DWF_ENOMEM && used == 0);
        {
            Scratch x({device, 0, 2, 1}, 3 * GB);
            code = 0;
            try { Scratch y({device, 0, 2, 1}, 3 * GB); } catch (const Error& e) { code = e.code; }
            CHECK(code == DWF_ENOMEM && used == 3 * GB);
        }
        CHECK(used == 3 * GB);
    }
    CHECK(used == 0 && live.empty());
    std::printf("done\n");
}
"""


@pytest.mark.skipif(HIPCC is None, reason="hipcc not found")
def test_scratch_pool_on_the_host(tmp_path):
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(PROGRAM)
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I" + CSRC, str(src), "-o",
                        str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout
    assert out == "done\n", out
