"""Device memory of a change of gauge field, on the host: upload_gauge of csrc/objects.cpp compiled against a counted
stand-in for the device allocator, its kernels not launched."""
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
#include <cstring>
#include <map>
static std::map<char*, size_t> live;
static size_t used = 0, most = 0;
static hipError_t fake_malloc(void** p, size_t n) {
    *p = std::calloc(1, n);
    live[(char*)*p] = n;
    used += n;
    most = used > most ? used : most;
    return hipSuccess;
}
static hipError_t fake_free(void* p) {
    used -= live[(char*)p];
    live.erase((char*)p);
    std::free(p);
    return hipSuccess;
}
static hipError_t fake_copy(void* d, const void* s, size_t n) {   // within one allocation, or it is an error
    auto it = live.upper_bound((char*)d);
    if (it == live.begin()) return hipErrorInvalidValue;
    --it;
    if ((char*)d + n > it->first + it->second) return hipErrorInvalidValue;
    std::memcpy(d, s, n);
    return hipSuccess;
}
#define hipMalloc(p, n) fake_malloc(p, n)
#define hipFree(p) fake_free(p)
#define hipMemset(p, v, n) (std::memset(p, v, n), hipSuccess)
#define hipMemcpy(d, s, n, k) fake_copy(d, s, n)
#define hipDeviceSynchronize() hipSuccess
#define hipStreamSynchronize(s) hipSuccess
#define hipGetLastError() hipSuccess
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#include "objects.cpp"
#include "blas.hip"

int main() {
    const int all[][4] = {{2, 2, 2, 2}, {4, 2, 2, 2}, {4, 4, 4, 6}, {6, 6, 2, 10}};
    for (const auto& dims : all) {
        dwf_lattice L;
        for (int mu = 0; mu < 4; ++mu) L.dims[mu] = dims[mu];
        L.antiperiodic_t = 1;
        L.V = (long)dims[0] * dims[1] * dims[2] * dims[3];
        L.Vh = L.V / 2;
        dwf::build_geometry(&L);
        std::vector<double> U((size_t)L.V * 72, 1.0);
        for (int k = 0; k < 2; ++k) {
            dwf::upload_gauge(&L, U.data(), false, nullptr);
            const size_t tables = L.nbr.bytes + L.lex_of_site_dev.bytes + L.links[0].bytes + L.links[1].bytes + L.links[2].bytes;
            std::printf("%ld: %zu %zu\n", L.V, most, tables);
        }
        most = 0;
    }
}
"""


@pytest.mark.skipif(HIPCC is None, reason="hipcc not found")
def test_host_links_need_no_device_memory_beyond_the_tables(tmp_path):
    src, exe = tmp_path / "links.hip", tmp_path / "links"
    src.write_text(PROGRAM)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O0", "-w", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-I" + CSRC, str(src), "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout.splitlines()
    assert len(out) == 8
    for line in out:
        most, tables = line.split(":")[1].split()
        assert int(most) == int(tables), line
