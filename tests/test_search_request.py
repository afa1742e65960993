"""Search requests of the sampling kernel for the recent policy (csrc/tns_layout.h): every lane must read the timestamp of
its own slot, wherever the slots lie in an edge array of up to 2^39 slots.  Built for the host; no GPU."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_17410_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include <initializer_list>
#include "tns_layout.h"
using namespace tns;
template <typename pos_t> int check(int64_t top) {
    for (int64_t base : {int64_t(0), int64_t(1) << 20, top / 3, top / 2, top - 200})
        for (int64_t slot0 = base; slot0 < base + 2 * kSlotsPerLine; ++slot0)
            for (int32_t n = 1; n <= 16; ++n)
                for (int closed = 0; closed < 2; ++closed) {
                    const SearchRequest r = make_request<pos_t>(slot0, n, 0.5f, closed);
                    if (request_slots(r) != n || request_closed(r) != (closed == 1) || r.t != 0.5f) return 2;
                    for (int32_t j = 0; j < 16; ++j)
                        if (request_word<pos_t>(r, j) != (uint64_t)slot_word(slot0 + (j < n ? j : n - 1))) {
                            std::printf("slot %lld of %d, lane %d\\n", (long long)slot0, n, j);
                            return 1;
                        }
                }
    return 0;
}
int main() { return WIDE ? check<int64_t>(kMaxEdgeOffset) : check<int32_t>((int64_t(1) << 31) / 32 * kSlotsPerLine); }
"""


@pytest.mark.parametrize("wide", [0, 1])
def test_every_lane_reads_its_slot(tmp_path, wide):
    src, exe = tmp_path / "requests.cpp", str(tmp_path / "requests")
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", f"-DWIDE={wide}", "-I", CSRC, str(src), "-o", exe])
    done = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout
