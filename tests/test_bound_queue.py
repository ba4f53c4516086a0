"""The order in which a wave of the search by bounds queues and drains what passes (csrc/bound_queue.h), replayed on the
CPU: whichever of a group's rows pass, the queue stays within its places, and nothing is lost."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1609_01882_amd", "csrc")

REPLAY = r"""
#include <cstdint>
#include <cstdio>
#include "bound_queue.h"

// One group: count[r] entries of register r, `fill` that wait.  Returns what waits then; *most the longest queue.
template <int GROUPS>
static int replay(const int *count, int fill, int *most)
{
    psc::queue_group<GROUPS>(
        [&](int t) { return count[3 * t] + count[3 * t + 1] + count[3 * t + 2] != 0; },
        [&](int r) { fill += count[r]; if (fill > *most) *most = fill; },
        [&]() { while (fill >= 64) fill -= 64; });
    return fill;
}
template <int GROUPS>
static int all()
{
    int most = 0, bad = 0;
    for (uint32_t rows = 0; rows < 1u << 16; ++rows) {  // every set of registers, full ones
        int count[16];
        for (int r = 0; r < 16; ++r) count[r] = rows >> r & 1u ? 64 : 0;
        for (int fill = 0; fill < 64; ++fill) bad += replay<GROUPS>(count, fill, &most) != fill;
    }
    uint32_t state = 1u;
    int fill = 0;
    for (int turn = 0; turn < 1000000; ++turn) {  // any number of lanes in each, group after group
        int count[16], sum = fill;
        for (int r = 0; r < 16; ++r) {
            state = state * 1664525u + 1013904223u;
            count[r] = state >> 28 < 6u ? 0 : (int)(state >> 20 & 0xffu) * 65 >> 8;
            sum += count[r];
        }
        fill = replay<GROUPS>(count, fill, &most);
        bad += fill != sum % 64;
    }
    printf("%d %d %d\n", most, psc::kQueuePlaces<GROUPS>, bad);
    return 0;
}
int main() { return all<HELD>(); }
"""


@pytest.mark.parametrize("groups,places", [(4, 640), (8, 1088)])
def test_queue_stays_within_its_places(tmp_path, groups, places):
    source, program = tmp_path / "replay.cpp", tmp_path / "replay"
    source.write_text(REPLAY)
    subprocess.run(["g++", "-O2", "-std=c++17", "-w", f"-DHELD={groups}", "-I", CSRC, str(source), "-o", str(program)], check=True)
    most, has, bad = map(int, subprocess.run([str(program)], check=True, capture_output=True, text=True).stdout.split())
    assert has == places and bad == 0
    assert most <= has, (most, has)
