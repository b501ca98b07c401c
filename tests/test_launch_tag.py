"""Tags of the arrival words (csrc/launch_tag.h), on the host: what a workspace can hold is not taken for arrivals of a launch."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_19505_amd", "csrc")

PROGRAM = r"""
#include "launch_tag.h"
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>
using namespace antkv;
// which arrivals merge, and how many workgroups have stored their part by then
static int merges_early(uint64_t word, uint64_t tag, uint32_t S)
{
    int early = 0, merges = 0;
    for (uint32_t stored = 1; stored <= S; ++stored) {
        if (arrivals_are_stale(word, tag, S)) word = tag;
        if ((word++ & kArrivalMask) + 1 == S) { ++merges; early += stored != S; }
    }
    return early || merges != 1;
}
int main()
{
    std::vector<uint64_t> tags(1 << 20);
    for (auto& t : tags) t = next_launch_tag();
    for (uint64_t t : tags)
        if (t & kArrivalMask) return std::puts("arrival bits"), 1;
    // pairs of small integers (index lists, counters, slice counts), of floats and of the same word twice
    for (int i = 0; i < 4096; ++i)
        for (uint32_t lo = 0; lo < 40; ++lo)
            for (uint32_t S : {2u, 8u, 32u, 1024u}) {
                const float f = (float)i / 64, g = (float)lo;
                uint32_t a, b;
                std::memcpy(&a, &f, 4);
                std::memcpy(&b, &g, 4);
                for (uint64_t w : {(uint64_t)i << 32 | lo, (uint64_t)a << 32 | b, (uint64_t)i << 32 | (uint32_t)i})
                    if (merges_early(w, tags[(i * 40 + lo) & 0xfffff], S)) return std::printf("%d %u %u\n", i, lo, S), 2;
            }
    // words of an earlier launch, and of this one replayed
    for (int i = 1; i < 1000; ++i)
        for (uint32_t S : {2u, 32u, 1024u})
            if (merges_early(tags[i - 1] + S, tags[i], S) || merges_early(tags[i] + S, tags[i], S) || merges_early(tags[i - 1] + 1, tags[i], S)) return 3;
    std::sort(tags.begin(), tags.end());
    if (std::adjacent_find(tags.begin(), tags.end()) != tags.end()) return std::puts("a tag twice"), 4;
    return 0;
}
"""


def test_arrival_words_of_any_content(tmp_path):
    src, exe = tmp_path / "tag.cpp", tmp_path / "tag"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stdout)
