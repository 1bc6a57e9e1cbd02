"""Every plan of the direct kernel has an instance, and every instance a plan: the plan's code, cut from the source and run on the host over
numbers of row tiles, column tiles and chunks around all its lines."""
import os
import re
import subprocess

from paper_2407_12075_amd import build as hip_build

_HOST = """
#include <cstdint>
#include <cstdio>
#include <initializer_list>
enum { TBN_F32 = 0, TBN_BF16 = 1 };
struct LinearArgs { int dt; int64_t M, in, p; };
constexpr int kMaxNT = %s, kChunkBytes = %s;
%s
%s
int main() {
    bool seen[2][kMaxNT + 1][9] = {};
    const int64_t far[] = {2000, 3072, 4096, 5000, 16384, 100000};
    for (int dt : {0, 1})
        for (int64_t chunks : {1, 12, 13, 216, 217, 1000})
            for (int r = 1; r <= 1606; ++r)
                for (int t = 1; t <= 76; ++t) {
                    const int64_t rows = r <= 1600 ? r : far[r - 1601], tiles = t <= 70 ? t : far[t - 71];
                    const int64_t in = chunks * (kChunkBytes / (dt == TBN_F32 ? 4 : 2));
                    const DirectPlan pl = plan(LinearArgs{dt, 32 * rows, in, 32 * tiles * in});
                    if (pl.wide) continue;   // two instances of their own
                    if (pl.nt < 1 || pl.nt > kMaxNT || pl.kw < 1 || pl.kw > 8) return 1;
                    seen[dt][pl.nt][pl.kw] = true;
                }
    int differ = 0, n = 0;
    for (int dt : {0, 1})
        for (int nt = 1; nt <= kMaxNT; ++nt)
            for (int kw : {1, 2, 4, 8}) {
                n += seen[dt][nt][kw];
                if (seen[dt][nt][kw] != planned(dt == TBN_F32, nt, kw)) { std::printf("%%d %%d %%d\\n", dt, nt, kw); ++differ; }
            }
    return differ || n != 18 ? 2 : 0;
}
"""


def test_instances_of_the_direct_kernel_are_those_that_are_planned(tmp_path):
    text = open(os.path.join(hip_build.CSRC, "tbn_linear_direct.hip")).read()
    plan = text[text.index("struct DirectPlan {"):text.index("}  // namespace", text.index("DirectPlan plan("))]
    planned = text[text.index("constexpr bool planned("):text.index("template <typename XT, int NT, int KW = 8>")]
    constant = lambda name: re.search(r"constexpr int(?:32_t)? " + name + r" = (\d+);", text).group(1)
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(_HOST % (constant("kMaxNT"), constant("kChunkBytes"), plan, planned))
    subprocess.run(["g++", "-O1", "-std=c++17", str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout
