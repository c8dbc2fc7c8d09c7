"""The bound of the outlier selection's writes, compiled for the host: what the kernel may find in its scratch words."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <initializer_list>
#include "rank_slot.h"
int main() {
    for (int32_t f : {0, 1, 64, 32768})
        for (int64_t r : {(int64_t)INT32_MIN, (int64_t)-2147483647, (int64_t)-64, (int64_t)-1, (int64_t)0, (int64_t)1, (int64_t)f - 1, (int64_t)f,
                          (int64_t)f + 1, (int64_t)INT32_MAX})
            if (rank_has_slot((int32_t)r, f) != (r >= 0 && r < f)) return 1;
    return 0;
}
"""


def test_only_ranks_inside_the_index_array_are_written(tmp_path):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2411_07762_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, str(src), "-o", str(exe)], check=True, timeout=60)
    assert subprocess.run([str(exe)], timeout=10).returncode == 0
    # and no subscript of idx by an unchecked rank is left in the kernel
    kernel = open(os.path.join(csrc, "smooth.hip")).read().split("void select_kernel", 1)[1].split("__global__", 1)[0]
    assert kernel.index("if (!rank_has_slot(r, f)) continue;") < kernel.index("idx[r] =") and kernel.count("idx[r]") == 1
