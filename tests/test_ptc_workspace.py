"""The learned preconditioner's workspace when the device has no memory for a larger lattice, on the host:
csrc/ptc.cpp compiled against a counted stand-in for the device allocator."""
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
#include <cstdlib>
static int budget = 1 << 30;   // allocations until the device is full
static hipError_t fake_malloc(void** p, size_t) {
    if (budget-- <= 0) return hipErrorOutOfMemory;
    *p = std::malloc(16);
    return hipSuccess;
}
#define hipMalloc(p, n) fake_malloc(p, n)
#define hipFree(p) (std::free(p), hipSuccess)
#define hipMemset(p, v, n) hipSuccess
#define hipMemsetAsync(p, v, n, st) hipSuccess
#define hipMemcpy(d, s, n, k) hipSuccess
#define hipGetLastError() hipSuccess
#include "ptc.cpp"
#include "scratch.cpp"
namespace dwf { int ptc_loss_blocks(long) { return 1; } }

int main() {
    for (int H : {1, 4})
        for (int full = 0; full < 12; ++full) {
            dwf_lattice small, large;
            small.V = 128; small.Vh = small.Vhp = 64;
            large.V = 1024; large.Vh = large.Vhp = 512;
            dwf_op a, b;
            a.Ls = b.Ls = 4;
            a.lat = &small;
            b.lat = &large;
            dwf_ptc M(H);
            M.reserve(&a, nullptr);
            budget = full;
            bool failed = false;
            try { M.reserve(&b, nullptr); } catch (const dwf::Error& e) { failed = e.code == DWF_ENOMEM; }
            budget = 1 << 30;
            M.reserve(&a, nullptr);
            bool ok = true;
            for (const dwf::DevBuf* x : {&M.hid, &M.y, &M.g, &M.lpartial, &M.d, &M.u, &M.w, &M.to, &M.tv})
                ok = ok && x->p;
            std::printf("H %d, full after %d: %s, then %s\n", H, full, failed ? "refused" : "accepted",
                        ok ? "complete" : "INCOMPLETE");
        }
}
"""


@pytest.mark.skipif(HIPCC is None, reason="hipcc not found")
def test_workspace_is_complete_after_a_failed_growth(tmp_path):
    """A call on a larger lattice fails for want of memory at each of its allocations in turn; the next call on the
    smaller lattice finds every buffer."""
    src, exe = tmp_path / "ws.cpp", tmp_path / "ws"
    src.write_text(PROGRAM)
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I" + CSRC, str(src), "-o",
                        str(exe), "-Wl,--unresolved-symbols=ignore-all"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(out) == 24 and sum("refused" in line for line in out) >= 16, out
    assert not [line for line in out if "INCOMPLETE" in line], out
