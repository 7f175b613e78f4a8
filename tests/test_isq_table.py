"""CPU check of the polynomials of the direct inverse square root (isq_table.h,
compiled here for the host): every plan, run as the kernels run it but in extended
precision, gives sqrt(x) Z(x) = 1 within half a unit of FP64's last place (plus
what rounding its coefficients to FP64 leaves) over its whole interval, the wide
plans of the 46-bit operands within 6e-15; the plans fit the program's length and
their ranges ascend."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include "isq_table.h"

int main() {
    for (int wide = 0; wide < 2; wide++) {
        const IsqTable tab = isq_build_table(wide);
        for (const IsqClass& k : tab.cls) {
            int products = 0;
            for (int s = 0; s < 3 && k.deg[s]; s++) {
                const bool last = s == 2 || !k.deg[s + 1];
                products += (s ? 1 : 0) + (k.deg[s] == 4 ? 2 : k.deg[s] == 6 ? 3 : 4) + (last ? 1 : s ? 2 : 1);
            }
            isq_ld worst = 0.0L;
            const int points = 20001;
            for (int i = 0; i < points; i++) {
                const isq_ld x = std::exp(-std::log((isq_ld)k.kappa) * i / (points - 1));
                isq_ld z = 0.0L, y = 0.0L;
                for (int s = 0; s < 3 && k.deg[s]; s++) {
                    const isq_ld X = ((s ? z * y : x) - (isq_ld)k.mid[s]) / (isq_ld)k.hw[s];
                    isq_ld w = 0.0L;
                    for (int j = k.deg[s]; j >= 0; j--) w = w * X + (isq_ld)k.b[s][j];
                    if (s == 0) { z = w; y = x * z; }
                    else { z += z * w; y += y * w; }
                }
                worst = std::max(worst, std::fabs(std::sqrt(x) * z - 1.0L));
            }
            std::printf("%d %.17g %d %.3Le\n", wide, k.kappa, products, worst);
        }
    }
}
"""


def test_composed_errors(tmp_path):
    src, exe = tmp_path / "table.cpp", tmp_path / "table"
    src.write_text(CHECK)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2308_03140_amd", "csrc"),
                           str(src), "-o", str(exe)])
    rows = [line.split() for line in subprocess.check_output([str(exe)]).decode().splitlines()]
    for wide in (0, 1):
        mine = [(float(r[1]), int(r[2]), float(r[3])) for r in rows if int(r[0]) == wide]
        assert mine == sorted(mine)
        for kappa, products, worst in mine:
            assert products <= 17, kappa
            assert worst <= (6e-15 if wide else 1.3e-16), (wide, kappa, worst)
