"""Every address of the dense MBD stage's symmetric product (k_mbd.hip, mfma_syrk_nt), on the CPU:
the function's own source, compiled for the host with the matrix instruction replaced by one that
returns its accumulator, runs for every lane on operands of exactly M x K elements under
AddressSanitizer, and every entry on or below the diagonal has to be stored exactly once.  K = 0 is
what exact forces have at n_max = 2 (no column of Tbar's product is left)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

HARNESS = r"""
#include <algorithm>
#include <cstddef>
#include <cstdio>
#include <type_traits>
#include <vector>
using std::min;
using std::max;
#define __device__
#define __forceinline__ inline
#define __syncthreads()
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x)
struct { int x; } threadIdx, blockDim;
template <typename V> void arrive(V&) {}
template <typename W> struct MfmaW {
    typedef W acc __attribute__((ext_vector_type(4)));
    static acc mma(W a, W b, acc c) { sink += a + b; return c; }   // (the operands are read)
    static int acc_row(int g, int q) { return sizeof(W) == 8 ? g + 4 * q : 4 * g + q; }
    static volatile W sink;
};
template <typename W> volatile W MfmaW<W>::sink = W(0);
@FUNCTION@
template <typename W>
static int check(int M, int K) {
    std::vector<W> A((size_t)M * K, W(1)), B((size_t)M * K, W(1));
    std::vector<int> seen((size_t)M * M, 0);
    blockDim.x = 512;
    for (threadIdx.x = 0; threadIdx.x < blockDim.x; ++threadIdx.x)
        mfma_syrk_nt<3, W>(M, K, A.data(), B.data(), K, [&](int r, int c, W) { seen[(size_t)r * M + c]++; });
    for (int r = 0; r < M; ++r)
        for (int c = 0; c < M; ++c)
            if (c <= r ? seen[(size_t)r * M + c] != 1 : seen[(size_t)r * M + c] > 1) return 1;
    return 0;
}
int main() {
    for (int M : {3, 15, 18, 48, 51, 99, 147})
        for (int K : {0, 4, 12, 16, 20, 36, 144, 180}) {
            std::printf("M %d K %d\n", M, K);
            std::fflush(stdout);
            if (check<double>(M, K) || check<float>(M, K)) return 1;
        }
    std::printf("ok\n");
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm toolchain")
def test_symmetric_product_reads_and_stores_in_bounds(tmp_path):
    with open(os.path.join(ROOT, "paper_2407_06409_amd", "csrc", "k_mbd.hip")) as fh:
        src = fh.read()
    m = re.search(r"template <int MR, typename W, typename ST>\n__device__ __forceinline__ void mfma_syrk_nt.*?\n}\n", src, re.S)
    assert m, "mfma_syrk_nt not found"
    cpp, exe = tmp_path / "syrk.cpp", tmp_path / "syrk"
    cpp.write_text(HARNESS.replace("@FUNCTION@", m.group(0)))
    subprocess.run([CLANG, "-std=c++17", "-O1", "-g", "-fsanitize=address", str(cpp), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    print(r.stdout[-300:], r.stderr[-3000:])
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-3000:]
