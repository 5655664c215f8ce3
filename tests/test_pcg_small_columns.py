"""The x neighbours that a lane of the one-workgroup Jacobi-PCG kernel reads from its 64 x 64 LDS array: inside the mesh's
row for every lane, the lanes beyond a mesh narrower than 64 nodes among them (their results are not used, but the
last one's right neighbour in the last row of 64 lies past the array).  The kernel's own text, evaluated on the host."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = """
#include <cstdio>
int main() {
    int bad = 0;
    for (int nx = 4; nx <= 64; ++nx)
        for (int x = 0; x < 64; ++x) {
            %s
            bad += xl < 0 || xl >= nx || xr < 0 || xr >= nx;
            if (x < nx) bad += xl != (x + nx - 1) %% nx || xr != (x + 1) %% nx;
        }
    std::printf("%%d\\n", bad);
}
"""


def test_neighbour_columns_stay_inside_the_row(tmp_path):
    src = open(os.path.join(ROOT, "paper_1902_09761_amd", "csrc", "kernels_pcg2d.hip")).read()
    m = re.findall(r"const int xl = [^;]*;", src)
    assert len(m) == 1
    cpp, exe = tmp_path / "columns.cpp", str(tmp_path / "columns")
    cpp.write_text(HARNESS % m[0])
    subprocess.run(["g++", "-std=c++17", str(cpp), "-o", exe], check=True)
    assert subprocess.run([exe], check=True, capture_output=True, text=True).stdout == "0\n"
