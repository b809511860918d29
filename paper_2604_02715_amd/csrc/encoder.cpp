// Code construction of the offline encoder of the compressed expert pool (host only; the loops over weights: encode_core.h).
//
// Paper Sec. 4.2 "Compressed GPU backend": only the exponent bits of the BF16 routed-expert
// weights are Huffman coded, offline; sign and mantissa bits are stored unchanged.  The
// block container is this library's own (documented in fluxmoe.h).
#include <algorithm>
#include <array>
#include <cstring>

#include "fluxmoe_internal.h"

namespace fluxmoe {

namespace {

struct Item {
    uint64_t weight;
    std::array<uint8_t, 256> count;   // how many leaves of each symbol the item contains
};

}  // namespace

// Package-merge: every used symbol contributes one leaf per level 1..lmax; from the deepest
// level upwards the items of a level (leaves plus the packages formed below) are sorted by
// weight and paired into packages for the level above; the 2(m-1) lightest items of level
// 1 are selected and a symbol's code length is the number of its leaves among them.
void limited_code_lengths(const uint64_t hist[256], uint32_t lmax, uint8_t lens[256]) {
    std::memset(lens, 0, 256);
    std::vector<int> used;
    for (int s = 0; s < 256; ++s)
        if (hist[s]) used.push_back(s);
    const size_t m = used.size();
    if (m == 0) return;
    if (m == 1) {
        lens[used[0]] = 1;
        return;
    }
    std::vector<Item> leaves(m);
    for (size_t i = 0; i < m; ++i) {
        leaves[i].weight = hist[used[i]];
        leaves[i].count.fill(0);
        leaves[i].count[used[i]] = 1;
    }
    auto by_weight = [](const Item& a, const Item& b) { return a.weight < b.weight; };
    std::stable_sort(leaves.begin(), leaves.end(), by_weight);
    std::vector<Item> packages, level;
    for (uint32_t depth = lmax; depth >= 1; --depth) {
        level.clear();
        level.resize(leaves.size() + packages.size());
        std::merge(leaves.begin(), leaves.end(), packages.begin(), packages.end(),
                   level.begin(), by_weight);
        if (depth == 1) break;
        packages.clear();
        for (size_t i = 0; i + 1 < level.size(); i += 2) {
            Item p;
            p.weight = level[i].weight + level[i + 1].weight;
            for (int s = 0; s < 256; ++s) p.count[s] = level[i].count[s] + level[i + 1].count[s];
            packages.push_back(p);
        }
    }
    const size_t take = 2 * (m - 1);
    for (size_t i = 0; i < take && i < level.size(); ++i)
        for (int s = 0; s < 256; ++s) lens[s] += level[i].count[s];
}

void canonical_codes(const uint8_t lens[256], uint16_t codes[256]) {
    std::memset(codes, 0, 256 * sizeof(uint16_t));
    uint32_t next = 0;
    uint32_t prev_len = 0;
    bool first = true;
    for (uint32_t len = 1; len <= 16; ++len) {
        for (int s = 0; s < 256; ++s) {
            if (lens[s] != len) continue;
            if (first) {
                next = 0;
                first = false;
            } else {
                next = (next + 1) << (len - prev_len);
            }
            codes[s] = static_cast<uint16_t>(next);
            prev_len = len;
        }
    }
}

}  // namespace fluxmoe
