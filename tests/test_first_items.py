"""The fixed first items of the attention launch's workgroups (host code): the
header's own functions, compiled and run over every small combination of chunk
items, decode items, decode-first workgroups and launch size.  Each kind's
fixed items are its lowest indexes, once each, so that the counters can deal
out the rest; decode-first workgroups start on decode items while there are any."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "mla_kernels.h"
#include <cstdio>
#include <vector>
int main() {
    for (int nc = 0; nc <= 9; ++nc)
        for (int nd = 0; nd <= 9; ++nd)
            for (int G = 1; G <= nc + nd && G <= 12; ++G)
                for (int D = 0; D <= G; ++D) {
                    const int fc = mla::first_chunk_items(nc, nd, D, G), fd = G - fc;
                    std::vector<int> seen(nc + nd, 0);
                    bool ok = fc >= 0 && fc <= nc && fd >= 0 && fd <= nd;
                    for (int b = 0; b < G && ok; ++b) {
                        const int it = mla::first_item(nc, nd, D, G, b);
                        ok = it >= 0 && it < nc + nd && (it < nc ? it < fc : it - nc < fd) && ++seen[it] == 1;
                        if (b < D && b < nd) ok = ok && it >= nc;
                        if (b >= D && b - D < nc) ok = ok && it < nc;
                    }
                    if (!ok) {
                        std::printf("chunk items %d, decode items %d, decode-first %d, workgroups %d\n", nc, nd, D, G);
                        return 1;
                    }
                }
    std::puts("ok");
}
"""


def test_every_fixed_item_once_and_lowest_first(tmp_path):
    cxx = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(cxx):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "first.cpp", tmp_path / "first"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2607_02043_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
