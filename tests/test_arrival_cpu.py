"""Counting of objective tiles (EXA_ARRIVAL, the text that the generated
kernels hold): one launch has one last tile, the last to arrive, and launches
that overlap, in any order, leave the counts fit for the next one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <random>
#include "paper_2608_16265_amd/csrc/exa_internal.h"
using namespace exa;

struct Counts {
    std::vector<unsigned> word;
    explicit Counts(long long n) : word(2 * count_words(n), 0) {}
    unsigned add(size_t i, unsigned w) {
        const unsigned b = word.at(i);
        word[i] += w;
        return b;
    }
};

// One tile's two steps (the count on its group's line, then the groups'): a
// launch's tiles can stop between them.
struct Tile {
    long long slot;
    int step = 0;
    bool last = false;
};

void advance(Counts& C, long long n, Tile& t) {
    const ExaArrival a = exa_arrival(t.slot, n);
    const size_t at = 2 * EXA_COUNT_AT(n);
    if (t.step == 0) {
        const bool full = exa_completes(C.add(at + 32 * a.line, a.weight), a.weight, a.bits);
        t.step = full && a.group_bits ? 1 : 2;
        t.last = full && !a.group_bits;
    } else {
        t.last = exa_completes(C.add(at, a.group_weight), a.group_weight, a.group_bits);
        t.step = 2;
    }
}

int main() {
    std::mt19937 rng(7);
    int bad = 0;
    for (long long n : {2, 3, 31, 32, 33, 63, 64, 65, 98, 489, 1024, 1025, 3907}) {
        Counts C(n);
        // close to where 32 bits wrap, after a whole number of launches
        for (unsigned& w : C.word) w = 0u - 4096u * 4u;
        for (int rep = 0; rep < 40; ++rep) {
            const int launches = rep % 2 ? 1 : 2 + rep % 3;  // every other time several overlap
            std::vector<Tile> t;
            for (int l = 0; l < launches; ++l)
                for (long long s = 0; s < n; ++s) t.push_back({s});
            std::vector<size_t> open(t.size());
            for (size_t i = 0; i < open.size(); ++i) open[i] = i;
            int lasts = 0;
            while (!open.empty()) {
                const size_t j = rng() % open.size();
                Tile& x = t[open[j]];
                advance(C, n, x);
                if (x.step < 2) continue;
                open[j] = open.back();
                open.pop_back();
                lasts += x.last;
                // alone: exactly the tile that arrives last
                if (launches == 1 && x.last != open.empty()) ++bad;
            }
            if (lasts != launches) ++bad;
        }
    }
    std::printf("%d\n", bad);
    return bad != 0;
}
"""


def test_counts_survive_overlapping_launches(tmp_path):
    src, exe = tmp_path / "arrival.cpp", tmp_path / "arrival"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", ROOT, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
