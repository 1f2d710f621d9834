"""The row launches of the sparse MBD stage (k_mbd_rows.hip) stay within 32 bits of work-items,
on the CPU: the source's own rule for the atoms of one set of launches, over neighbourhoods of up
to 32,768 sites, any number of column chunks and up to 10^7 atoms."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

HARNESS = r"""
#include <algorithm>
#include <cstdio>
@FUNCTION@
int main() {
    for (int nk : {1, 2, 64, 91, 306, 2450, 6600, 16500, 31000, 32768})
        for (int chunks : {1, 2})
            for (int n : {1, 7, 8, 9, 513, 6401, 100003, 10000000}) {
                const long long parts = ((nk + 1) / 3 + 1) * chunks / 4 + 1, threads = std::max(1024ll, 256 * parts);
                const int most = rows_atoms_per_launch(n, threads);
                if (most < 1 || most > n) return 1;
                if (most < n && most % 8) return 2;
                if ((most + 7) / 8 * 8 * threads > 0xffffffffll) return 3;
            }
    std::printf("ok\n");
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm toolchain")
def test_row_launches_fit_32_bits(tmp_path):
    with open(os.path.join(ROOT, "paper_2407_06409_amd", "csrc", "k_mbd_rows.hip")) as fh:
        src = fh.read()
    m = re.search(r"static int rows_atoms_per_launch.*?\n}\n", src, re.S)
    assert m, "one launch takes any number of atoms"
    # every launch of a kernel over (atom, part) is sized by the atoms of its set
    assert not re.search(r"dim3\(\s*8u?\s*\*", src) and src.count("for (int first = 0; first < all.n; first += most)") == 1
    cpp, exe = tmp_path / "launch.cpp", tmp_path / "launch"
    cpp.write_text(HARNESS.replace("@FUNCTION@", m.group(0)))
    subprocess.run([CLANG, "-std=c++17", str(cpp), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)
