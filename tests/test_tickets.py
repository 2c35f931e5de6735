"""The tickets by which a launch finds the writer of a head's last record (csrc/ticket.h), compiled for the
host: whatever order the steps of any number of launches are taken in, the word ends at zero, and a launch
that runs alone has exactly one last writer, the one that steps last."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_10516_amd", "csrc")

SOURCE = r"""
#include <stdio.h>
#include <algorithm>
#include <random>
#include <vector>
#include "ticket.h"
int main() {
    std::mt19937 rng(7);
    auto steps_of = [&](int P, std::vector<uint32_t>& s) { for (int r = 0; r < P; ++r) s.push_back(ticket_step(r, P)); };
    uint32_t word = 0u;
    for (int round = 0; round < 4000; ++round) {
        // a few launches at once, of 1 to 40 records, their steps in any order
        std::vector<uint32_t> s;
        for (int l = 1 + (int)(rng() % 4); l > 0; --l) steps_of(1 + (int)(rng() % 40), s);
        std::shuffle(s.begin(), s.end(), rng);
        for (uint32_t x : s) word += x;
        if (word != 0u) { printf("round %d: the word is left at %u\n", round, word); return 1; }
        // then one alone
        std::vector<uint32_t> one;
        const int P = 1 + (int)(rng() % (round % 100 ? 40 : 100000));
        steps_of(P, one);
        std::shuffle(one.begin(), one.end(), rng);
        for (int i = 0; i < P; ++i) {
            const bool last = ticket_last(word, one[i]);
            word += one[i];
            if (last != (i == P - 1)) { printf("%d records: step %d is %d\n", P, i, (int)last); return 1; }
        }
    }
    printf("ok\n");
    return 0;
}
"""


def test_tickets_come_back_to_zero_and_name_one_last_writer(tmp_path):
    src, exe = tmp_path / "tickets.cpp", tmp_path / "tickets"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True,
                   timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
