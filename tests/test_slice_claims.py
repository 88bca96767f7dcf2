"""The places that blocks get in the emission's slice list (fg_slices.h), compiled
for the host: whatever the order in which the blocks add to the counter, every
entry that is read was written by its owner, and a block's slices are
listed all or not at all."""
import os
import subprocess


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "fg_slices.h"
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

// Blocks want w[b] slices each. A block's two steps are its addition to the counter
// and its writes; the writes use what the addition returned, so they may come at any
// later time. All orders of additions, writes in that order and in reverse.
static int check(const std::vector<uint64_t>& w, uint64_t cap)
{
    std::vector<int> order(w.size());
    for (size_t i = 0; i < order.size(); i++) order[i] = (int)i;
    do {
        uint64_t counter = 0;
        std::vector<fgs::Claim> c(w.size());
        for (int b : order) {
            c[b] = fgs::claim(counter, w[b], cap);
            counter += w[b];
        }
        std::vector<std::pair<int, uint64_t>> list(cap, {-2, 0});  // -2: never written, -1: empty
        std::vector<int> written(cap, 0);
        for (int b : order)
            for (uint64_t k = c[b].first; k < c[b].last; k++) {
                if (k >= cap) return 1;  // out of the list
                written[k]++;
                list[k] = c[b].listed ? std::make_pair(b, k - c[b].first + 1) : std::make_pair(-1, (uint64_t)0);
            }
        std::vector<uint64_t> seen(w.size(), 0);
        for (uint64_t k = 0; k < fgs::entries(counter, cap); k++) {
            if (written[k] != 1) return 2;  // unwritten, or two owners
            if (list[k].first >= 0) seen[list[k].first] |= 1ull << list[k].second;
        }
        uint64_t sum = 0;
        for (size_t b = 0; b < w.size(); b++) {
            sum += w[b];
            const uint64_t all = ((1ull << w[b]) - 1) << 1;
            if (seen[b] != (c[b].listed ? all : 0)) return 3;  // part of a block listed
        }
        if (sum <= cap)
            for (auto& x : c)
                if (!x.listed) return 4;  // refused although everything fits
    } while (std::next_permutation(order.begin(), order.end()));
    return 0;
}

int main()
{
    for (uint64_t cap = 1; cap <= 8; cap++)
        for (uint64_t a = 1; a <= 6; a++)
            for (uint64_t b = 1; b <= 6; b++)
                for (uint64_t c = 1; c <= 6; c++)
                    for (uint64_t d = 1; d <= 3; d++)
                        if (int rc = check({a, b, c, d}, cap)) {
                            std::printf("cap %d claims %d %d %d %d: fault %d\n", (int)cap, (int)a, (int)b, (int)c, (int)d, rc);
                            return 1;
                        }
    // the counter past 32 bits, and claims that end at the largest value
    if (fgs::claim(1ull << 33, 1, 1ull << 21).listed || fgs::claim(0, ~0ull, 5).listed) return 2;
    if (fgs::claim(~0ull, ~0ull, 5).first != 5 || fgs::entries(~0ull, 5) != 5) return 3;
    std::printf("ok\n");
    return 0;
}
"""


def test_claims_in_every_order(tmp_path):
    src, exe = tmp_path / "claims.cpp", tmp_path / "claims"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2603_23891_amd", "csrc"), "-o",
                        str(exe), str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
