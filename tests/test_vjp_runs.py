"""Index arithmetic of the x face VJP on the CPU: the cells a wave's 64 faces
touch form one run of the padded plane, every face's six-cell stencil lies in
the run, the run fits the LDS window the host sizes for it, and the runs of
every second wave share no cell; for three and four ghost layers, rows shorter
and longer than a wave."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")

SOURCE = r"""
#include "xf_common.hpp"
#include <cstdio>
#include <initializer_list>
int main() {
    long long bad = 0, faces = 0;
    for (int gx : {3, 4})
        for (int nx = gx; nx <= 200; ++nx)
            for (int ny : {1, 4, 7, 40}) {
                xf::Geo g{};
                g.nx = nx; g.ny = ny; g.gx = gx;
                g.sy = nx + 2 * gx;
                const long long nf = (nx + 1ll) * ny;
                const int W = xf::vjp_x_run(g);
                long long end2 = -1, end1 = -1;   // ends of the runs two and one waves back
                for (long long f0 = 0; f0 < nf; f0 += 64) {
                    const long long fl = f0 + 63 < nf ? f0 + 63 : nf - 1;
                    const long long base = xf::vjp_x_first(g, f0), span = xf::vjp_x_first(g, fl) - base + 6;
                    bad += span > W || base < end2;
                    end2 = end1;
                    end1 = base + span;
                    for (long long f = f0; f <= fl; ++f, ++faces) {
                        // interior cell 0 of the row lies at gx; the stencil of face i starts at cell i - 3
                        const long long row = f / (nx + 1), i = f % (nx + 1), off = row * g.sy + gx + i - 3 - base;
                        bad += off < 0 || off + 6 > span;
                    }
                }
            }
    std::printf("%lld %lld\n", bad, faces);
}
"""


def test_stencils_lie_in_their_waves_run(tmp_path):
    src, exe = tmp_path / "runs.hip", tmp_path / "runs"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_2403_05910_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    bad, faces = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert faces > 10 ** 6
    assert bad == 0
