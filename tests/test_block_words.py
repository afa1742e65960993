"""Where a block's slots lie, from one division per block (BlockWords in csrc/tns_layout.h), against a division per slot: every
position in a line, every part of the 39-bit slot index, the records' other bits set and clear.  Built for the host; no GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_17410_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include <initializer_list>
#include "tns_layout.h"
using namespace tns;
int main() {
    const int32_t most = (1 << 24) - 1;      // size of a block
    uint64_t random = 1;
    auto check = [&](int64_t off) {
        for (int32_t size : {1, most}) {
            for (int holes = 0; holes < 2; ++holes) {
                const BlockWords words(make_rec(0.5f, 1.5f, off, size, holes));
                random = random * 6364136223846793005ull + 1442695040888963407ull;
                for (int32_t i : {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 19, 20, 21, (int32_t)(random >> 40), most - 1, most})
                    if ((int64_t)(words.base + words.words_to(i)) != slot_word(off + i) || words.base % 32 || words.at >= (uint32_t)kSlotsPerLine) {
                        std::printf("slot %d of the block at %lld\\n", i, (long long)off);
                        return false;
                    }
            }
        }
        return true;
    };
    for (int64_t off = 0; off < 3000; ++off)
        if (!check(off)) return 1;
    for (int64_t high = 1; high < 128; ++high)
        for (int64_t near = -25; near < 25; ++near)
            if (!check((high << 32) + near)) return 1;
    for (int64_t off = kMaxEdgeOffset - 3000; off <= kMaxEdgeOffset; ++off)
        if (!check(off)) return 1;
    for (int n = 0; n < 200000; ++n) {
        random = random * 6364136223846793005ull + 1442695040888963407ull;
        if (!check((int64_t)(random >> 8) % (kMaxEdgeOffset + 1))) return 1;
    }
    return 0;
}
"""


def test_slots_of_a_block(tmp_path):
    src, exe = tmp_path / "words.cpp", str(tmp_path / "words")
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", exe])
    done = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout
