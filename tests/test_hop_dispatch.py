"""Which kernel a hop launch takes, checked on the host: the launchers' own source is compiled with its kernel
launches replaced by a record of the kernel's name and template arguments (no GPU, nothing is launched)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_14454_amd", "csrc")
HIPCC = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)),
             None)
pytestmark = pytest.mark.skipif(HIPCC is None, reason="hipcc not found")

RECORD = r"""
#include <cstdio>
#include "hop_tile.h"
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, ...) std::printf("  launch %s | %s\n", #kernel, __PRETTY_FUNCTION__)
#undef hipGetLastError
#define hipGetLastError() hipSuccess
"""


def _run(tmp_path, body, *flags):
    src, exe = tmp_path / "dispatch.hip", tmp_path / "dispatch"
    src.write_text(RECORD + body)
    cmd = [HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O0", "-w", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + CSRC, *flags, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout.splitlines()


def test_small_lattice_form_takes_only_its_own_launches(tmp_path):
    """Every pre-mix mode with every epilogue kind, -1 (none compiled) included: the small-lattice form launches
    the kernel of exactly that pair, or declines and launches nothing."""
    out = _run(tmp_path, r"""
#include "hop_few.hip"
namespace dwf { int hop_grid_blocks(long Vh) { return (int)((Vh + 15) / 16); } }
int main() {
    for (int Ls : {2, 4, 5, 8, 9, 16})
        for (int pm = -1; pm <= 3; ++pm)
            for (int ek = -2; ek <= 9; ++ek) {
                dwf::HopParams P{};
                P.Vh = 128;
                P.Ls = Ls;
                P.pre_mode = pm;
                std::printf("case %d %d %d\n", pm, ek, Ls);
                std::printf("  taken %d\n", (int)dwf::launch_hop_few(P, 1, ek, nullptr));
            }
}
""")
    forms = {0: (1, 2, 3, 4, 5, 6, 7), 1: (1, 4), 2: (1, 4)}   # epilogue kinds by pre-mix mode
    cases, pair = [], None
    for line in out:
        w = line.split()
        if w[0] == "case":
            pair = tuple(int(v) for v in w[1:])
            cases.append([pair, [], None])
        elif w[0] == "launch":
            cases[-1][1].append(line.split("|")[1])
        else:
            cases[-1][2] = int(w[1])
    assert len(cases) == 6 * 5 * 12
    for (pm, ek, Ls), launches, taken in cases:
        if ek in forms.get(pm, ()) and not (ek == 7 and Ls <= 4):   # 7 forms alpha: never asked for at Ls <= 4
            assert taken == 1 and len(launches) == 1, (pm, ek, launches)
            assert f"PM = {pm}, EK = {ek}," in launches[0], (pm, ek, launches)
        else:
            assert taken == 0 and not launches, (pm, ek, launches)


@pytest.mark.parametrize("define", ["DWF_HOP_EK=1", "DWF_HOP_EK=0"])
def test_update_that_forms_alpha_has_its_kernel(tmp_path, define):
    """The last hop of a CG step with the step length formed in it (HopParams::sum), which small solves use in every
    precision: the launch finds the kernel that does this, with any definition of the former switch DWF_HOP_EK."""
    out = _run(tmp_path, r"""
#include "hop.hip"
namespace dwf { bool launch_hop_few(const HopParams&, int, int, hipStream_t) { return false; } }
int main() {
    using namespace dwf;
    double some[1];
    for (int Ls = 5; Ls <= 16; ++Ls)
        for (int kind : {ST_F64, ST_F32, ST_BF16}) {
            HopParams P{};
            P.Vh = 128;
            P.Ls = Ls;
            P.loc = P.locmix = P.upd = P.partial = P.scal = some;
            P.sum = some;
            P.nsum = 8;
            P.reduce = 3;
            std::printf("case %d %d\n", Ls, kind);
            try {
                launch_hop(kind, P, 1, nullptr);
            } catch (const Error& e) {
                std::printf("  refused %s\n", e.msg.c_str());
            }
        }
}
""", "-D" + define)
    assert len(out) == 2 * 12 * 3 and not [line for line in out if "refused" in line], out
    for line in out[1::2]:
        assert "hop_mfma_kernel" in line and "PM = 0, EK = 7" in line, line
