"""Division by a number fixed on the host (FastDiv) and the splitting of linear
indices on the CPU: quotients at and beside every multiple's edge up to 2^31 for
divisors over their whole range, and the 32-bit split against the 64-bit one
(grids of 2^31 cells and more take the latter) and against plain division."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")

SOURCE = r"""
#include "xf_common.hpp"
#include <cstdio>
#include <random>
int main() {
    std::mt19937_64 rng(1);
    long long bad = 0, tried = 0;
    const unsigned long long top = (1ull << 31) - 1;   // the largest n
    auto quotient = [&](const xf::FastDiv &f, unsigned long long d, unsigned long long n) {
        if (n > top) return;
        bad += f.of((unsigned)n) != n / d;
        ++tried;
    };
    auto divisor = [&](unsigned long long d) {
        xf::FastDiv f;
        f.set((long long)d);
        const unsigned long long k = top / d;   // the last multiple
        for (unsigned long long q : {0ull, 1ull, 2ull, k / 2, k - (k > 0), k})
            for (int e = -1; e <= 1; ++e) quotient(f, d, q * d + e);
        quotient(f, d, top);
        for (int r = 0; r < 8; ++r) quotient(f, d, rng() & top);
    };
    for (unsigned long long d = 1; d <= 70000; ++d) divisor(d);
    for (int l = 17; l <= 30; ++l)
        for (long long e = -2; e <= 2; ++e) divisor((1ull << l) + e);
    for (int r = 0; r < 100000; ++r) divisor(1 + (rng() & top) % top);
    divisor(top);
    // splitting: q over (a, b, c)
    for (int r = 0; r < 200000; ++r) {
        const int a = 1 + rng() % 65541, b = 1 + rng() % (r % 2 ? 40 : 65541);
        xf::Geo g{};
        xf::FastDiv da, db;
        da.set(a);
        db.set(b);
        long long q = r % 3 == 0 ? (long long)(rng() & top) : (long long)a * b * (rng() % 50) + rng() % 3 - 1;
        if (q < 0) q = 0;
        int x[2], y[2], z[2];
        for (int small = 0; small < 2; ++small) {
            if (small && q > (long long)top) continue;
            g.small = small;
            xf::split3(g, q, a, b, da, db, x[small], y[small], z[small]);
            bad += x[small] != q % a || y[small] != q / a % b || z[small] != q / a / b;
            ++tried;
        }
    }
    std::printf("%lld %lld\n", bad, tried);
}
"""


def test_quotients_and_splits(tmp_path):
    src, exe = tmp_path / "split.hip", tmp_path / "split"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_2403_05910_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    bad, tried = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert tried > 10 ** 6
    assert bad == 0
