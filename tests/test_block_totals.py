"""Who hands out the sums of block_totals (kernels_common.h).  The kernel that announces them to other workgroups does
so from thread 0 (a release fence and an atomic), and a wave waits for the stores of its own lanes only, so every
sum has to be stored by the first wave.  The function's own text, run on the host one thread after the other."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = """
#include <cstdio>
#define __device__
#define __forceinline__ inline
struct { unsigned x; } threadIdx;
static void __syncthreads() {}
template <int NV, typename F> void wave_sums(double (&)[NV], F&&) {}   // the waves' sums are in lds already
%s
template <int NV> int run() {
    double lds[4 * NV], v[NV];
    int calls[NV] = {}, bad = 0;
    for (int i = 0; i < 4 * NV; ++i) lds[i] = 1 + i / NV + 10.0 * (i %% NV);
    for (unsigned t = 0; t < 256; ++t) {
        threadIdx.x = t;
        block_totals<NV>(v, lds, [&](int i, double s) {
            calls[i]++;
            bad += t >= 64 || s != 10.0 + 40.0 * i;
        });
    }
    for (int i = 0; i < NV; ++i) bad += calls[i] != 1;
    return bad;
}
int main() { std::printf("%%d %%d %%d %%d %%d\\n", run<1>(), run<17>(), run<63>(), run<64>(), run<65>()); }
"""


def test_every_sum_is_stored_by_the_first_wave(tmp_path):
    src = open(os.path.join(ROOT, "paper_1902_09761_amd", "csrc", "kernels_common.h")).read()
    m = re.search(r"template <int NV, typename F>\n__device__ __forceinline__ void block_totals\(.*?\n}\n", src, re.S)
    assert m
    cpp = tmp_path / "totals.cpp"
    cpp.write_text(HARNESS % m.group(0))
    exe = str(tmp_path / "totals")
    subprocess.run(["g++", "-std=c++17", str(cpp), "-o", exe], check=True)
    assert subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split() == ["0"] * 5
