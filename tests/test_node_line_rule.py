"""Which node lines are read without the non-temporal hint (csrc/tns_layout.h): small tables and skewed degrees, but not lists that
are long everywhere.  Built for the host; no GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_17410_amd", "csrc")

PROGRAM = """
#include "tns_layout.h"
int main() {
    const int64_t n = int64_t(1) << 20, small = int64_t(1) << 17;
    auto stay = tns::node_lines_stay;
    if (!stay(small, small, 0, 0) || !stay(small, 256 * small, 0, 3 * small)) return 1;      // small tables, one or many
    if (stay(small + 1, small + 1, 0, small) || stay(n, n, n / 16 - 1, n)) return 2;         // short lists
    if (!stay(n, n, n / 16, 2 * n) || !stay(n, n, 40 * n, 6 * n)) return 3;                  // few long lists
    if (stay(n, n, 9 * n, 8 * n) || stay(n, n, 30 * n, 15 * n)) return 4;                    // long lists everywhere
    return 0;
}
"""


def test_long_lists_everywhere_are_no_skew(tmp_path):
    src, exe = tmp_path / "rule.cpp", str(tmp_path / "rule")
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", exe])
    assert subprocess.run([exe], timeout=60).returncode == 0
