"""The intervals of a balanced leaf launch (TapeWalk), walked on the host: over
random tables every block of every group is hashed exactly once, a group across
a boundary by two neighbouring waves that agree on the cut, whatever the
lengths, the wave counts and the set-up a group is given."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_23938_amd", "csrc")
SOURCE = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "balance.h"

static uint64_t state = 7;
static uint64_t rnd(uint64_t below) {  // xorshift64*
    state ^= state >> 12; state ^= state << 25; state ^= state >> 27;
    return (state * 2685821657736338717ull >> 16) % below;
}
#define CHECK(x) do { if (!(x)) { printf("%s, table %d\n", #x, table); return 1; } } while (0)

int main() {
    for (int table = 0; table < 20000; ++table) {
        const uint32_t waves = 4 * (1 + (uint32_t)rnd(12)), setup = (uint32_t)rnd(5);
        const uint64_t full = rnd(40), tails = rnd(3) == 0 ? 0 : rnd(80), blocks = 1 + rnd(rnd(2) ? 9 : 600);
        if (full + tails == 0) continue;
        std::vector<uint64_t> head(tails + 2), len(full + tails);
        uint64_t at = 0, bound = full ? blocks : 1 + rnd(600);
        head[0] = full;
        for (uint64_t g = 0; g < full; ++g) { len[g] = blocks; at += setup + blocks; }
        for (uint64_t g = 0; g < tails; ++g) {  // not rising, as the table is sorted
            if (rnd(3) == 0) bound = 1 + rnd(bound);
            head[1 + g] = at;
            len[full + g] = bound;
            at += setup + bound;
        }
        head[1 + tails] = at;
        hv::Tape t = {head.data(), nullptr, nullptr, blocks + setup, setup, waves};
        std::vector<uint32_t> upto(full + tails, 0), by(full + tails, 0), done(full + tails, 0);
        uint64_t longest = 0;
        for (uint64_t g = 0; g < full + tails; ++g) if (len[g] + setup > longest) longest = len[g] + setup;
        for (uint32_t w = 0; w < waves; ++w) {  // in the order of dispatch: the saved states come from before
            hv::TapeWalk walk(t, 64 * (full + tails) - rnd(tails ? 64 : 1), w);
            hv::Piece p;
            uint64_t length = 0;
            for (int n = 0; walk.next(&p); ++n) {
                CHECK(p.group < full + tails);
                if (!p.last) {
                    CHECK(n == 0);  // at its interval's start: the states are there first
                    CHECK(p.from == 0 && p.to < len[p.group] && p.to % 2 == 0);
                    upto[p.group] = p.to;
                    by[p.group] = w + 1;
                } else {
                    CHECK(p.to == len[p.group] && done[p.group]++ == 0);
                    if (p.from > 0) CHECK(by[p.group] == w && upto[p.group] == p.from);
                    else CHECK(upto[p.group] == 0);
                }
                length += p.to - p.from;
            }
            CHECK(length <= (at + waves - 1) / waves + 1 || length <= longest + 1);  // a cut lies on an even block
        }
        for (uint64_t g = 0; g < full + tails; ++g) CHECK(done[g] == 1);
    }
    printf("walked\n");
    return 0;
}
"""


def test_every_block_once(tmp_path):
    src = tmp_path / "walk.cpp"
    src.write_text(SOURCE)
    exe = tmp_path / "walk"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-std=c++17",
                    "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.stdout.strip() == "walked", r.stdout
