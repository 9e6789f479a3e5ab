"""Probes of the small update's hash table (csrc/edge_hash.h, linear probing, at most half full) for regular batches,
counted in a CPU program."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_05396_amd", "csrc")

PROGRAM = r"""
#include "edge_hash.h"
#include <stdio.h>
#include <vector>
int main() {
    const unsigned strides[] = {1, 2, 3, 64, 511, 512, 513, 600, 1000, 1024, 2047, 2048, 2049, 2584, 4096, 6144, 6765, 10946, 17711, 28657, 46368,
                                65536, 75025, 121393, 196418, 317811, 514229, 832040, 1000000, 1048576, 1346269, 2095104};
    int bad = 0;
    for (unsigned b : {8u, 100u, 512u, 600u, 1024u})
        for (unsigned stride : strides)
            for (unsigned first : {0u, 1u, 777u}) {
                unsigned slots = 2;
                while (slots < 2 * b) slots *= 2;
                std::vector<int> table(slots, -1);
                unsigned most = 0, sum = 0;
                for (unsigned i = 0; i < b; ++i) {
                    unsigned slot = edge_hash(first + i * stride) & (slots - 1), probes = 1;
                    while (table[slot] >= 0) slot = (slot + 1) & (slots - 1), ++probes;
                    table[slot] = (int)i;
                    sum += probes;
                    if (probes > most) most = probes;
                }
                // a random function at half load: 1.5 on average, below 30 at the longest (log of 1 024 entries)
                if (most > 40 || sum > 2 * b + 20) printf("b %u stride %u first %u: %u probes at most, %u in all\n", b, stride, first, most, sum), bad = 1;
            }
    return bad;
}
"""


def test_regular_batches_probe_like_random_ones(tmp_path):
    (tmp_path / "h.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-isystem", "/opt/rocm/include", "-o",
                    str(tmp_path / "h"), str(tmp_path / "h.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "h")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
