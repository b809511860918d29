// Launch plan of the expert FFN: which kernels, tiles and K splits a call takes, and how its scratch is laid out.
// Host arithmetic only, without HIP, so that the rules can be tested on their own.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>

namespace fluxmoe {

// Batches with more pairs than this are counted and scattered by one workgroup per kRouteChunkPairs pairs
// around the single workgroup that scans the experts.  Microseconds, one workgroup / several (three launches), 8 to 512
// experts: 12288 pairs 17.3 / 18.3, 16384 20.7 / 18.7, 32768 35.4 / 20.6, 163840 - / 31.
constexpr uint32_t kRouteChunkThreshold = 14336;
constexpr uint32_t kRouteChunkPairs = 4096;
// Calls of up to this many pairs on strip kernels have no grouping kernel: the first product's workgroups group the pairs.
constexpr uint32_t kFewPairs = 64;
// Partial sums of a last round (last_round_kernel): at most seven blocks of a super-tile's 32 tiles of 256 x 256.
constexpr uint64_t kTailBytes = 7ull * 32 * 256 * 256 * 4;
// Row tiles a call may have (the z dimension of the strip kernels' grid).
constexpr uint32_t kMaxRowTiles = 65535;

#if defined(__HIPCC__)
#define FLUXMOE_HD __host__ __device__
#else
#define FLUXMOE_HD
#endif

// Splitting the first product's K pays while the row tiles leave CUs without work.  The plan goes by the mean of what an expert
// gets; skewed routing makes more tiles, and then every split is another round.  So the kernels, which see the count,
// decide: up to split_tiles row tiles the plan's ksplit1 splits work; past them a single one, and with 256 x 256 tiles the
// number with the least tiled_cost.  Microseconds per call, always ksplit1 / decided (never split): 1024 tokens that all take
// the two resident of 8 experts of H 4096 F 3584 266 / 212 (206), the four resident of 160 of H 5120 F 1536 480 / 380 (340),
// 4096 tokens on the eight resident of 128 of H 2048 F 512 445 / 344 (335); 20 experts of H 5120 F 384, 410 rows each 250 / 230
// (236), where the model sees a second round that the tile count does not show.
struct SplitShape {
    uint32_t H, F, n_cus;
};
// Nanoseconds of the first product in 256 x 256 tiles with K split k ways: 3 us to start a tile, 1.4 us a step of 64 k, partial
// sums at 10 TB/s.  (Super-tile of 4 x 8 tiles, split) pairs are dealt to the 8 XCDs; the fullest XCD counts.
FLUXMOE_HD inline float tiled_cost(const SplitShape& s, uint32_t n_tiles, uint32_t rows, uint32_t k) {
    const uint32_t n_ct = (s.F + 127) / 128, per_xcd = s.n_cus / 8 ? s.n_cus / 8 : 1;
    const uint32_t pairs = ((n_tiles + 3) / 4) * ((n_ct + 7) / 8) * k;
    const uint32_t tiles = (pairs + 7) / 8 * (n_tiles < 4 ? n_tiles : 4u) * (n_ct < 8 ? n_ct : 8u);
    const float steps = float((s.H / 64 + k - 1) / k);
    return float((tiles + per_xcd - 1) / per_xcd) * (steps * 1400.f + 3000.f) + (k > 1 ? 4500.f + float(k) * float(rows) * float(s.F) * 16.f / 10000.f : 0.f);
}

// The last round of a second product in 256 x 256 tiles.  Super-tiles of 4 x 8 tiles are dealt to the 8 XCDs in turn; where the last
// round has four of them at most, K of each is split over as many XCDs as there are for one, and last_round_kernel adds the parts up.
// 8 experts of H 4096 F 14336, 4096 tokens, top-2 (18 super-tiles, two XCDs ran a third round while six had nothing to do): 916 -> 840 us
// with the sums and route_order_kernel.
struct LastRound {
    uint32_t first, parts;       // first super-tile of the round, parts of K
};
FLUXMOE_HD inline LastRound last_round(uint32_t supers) {
    const uint32_t rest = supers % 8u;
    return LastRound{supers - rest, rest == 1 ? 8u : (rest == 2 ? 4u : (rest == 3 || rest == 4 ? 2u : 1u))};
}
// From this F on it pays.  Microseconds a call, whole / split last round, two experts, one to four super-tiles left and five (whole, but for the
// launches): H 2048 F 2112 324 / 318, 342 / 343, 358 / 358, 385 / 388, 427 / 434; F 3072 411 / 395, 411 / 394, 471 / 454, 497 / 494, 538 / 546; F 4096
// 513 / 481, 514 / 488, 586 / 560, 617 / 598, 659 / 669; F 7168 870 / 796, 858 / 794, 939 / 886, 1015 / 975, 1090 / 1099.
constexpr uint64_t kLastRoundF = 3072;
// Whether a call of `pairs` pairs launches what a split last round needs.  Only the device knows the number of row tiles; where the round turns out
// whole, the two launches are 8 us for nothing (8 experts of H 4096 F 3584, 936 rows each 661 / 668).  So the gain, 3/8 of what the round's length
// promises, has to cover them, counting two thirds on rows dealt evenly and one on any number of tiles that a routing can make.
inline bool last_round_pays(uint64_t pairs, uint64_t mapped, uint64_t E, uint64_t H, uint64_t F) {
    const uint64_t act = mapped ? std::min(mapped, E) : E, rows = pairs * act / E, n_sn = ((H + 255) / 256 + 7) / 8;
    if (rows == 0) return false;
    const uint64_t experts = std::min(act, rows), least = (rows + 255) / 256, most = (rows + 255 * experts) / 256;
    const double round_us = 3.0 + 1.4 * double((F + 63) / 64);
    const auto gain = [&](uint64_t tiles) { return 0.375 * round_us * (1.0 - 1.0 / last_round(uint32_t((tiles + 3) / 4 * n_sn)).parts); };
    double any = 0.0;
    for (uint64_t n = least; n <= most; ++n) any += gain(n);
    const uint64_t even = experts * (((rows + experts - 1) / experts + 255) / 256);
    return (2.0 * gain(even) + any / double(most - least + 1)) / 3.0 > 8.0;
}

struct FfnPlan {
    bool tiled, halves, g1_xcd;
    // few: the first product's workgroups group the pairs.  few_splits: gemm2_few_kernel runs with as many K splits, which ksplit tells too.
    // few_fused: it also adds up the first product's partial sums, which then lie at off_part behind y
    bool few, few_fused;
    bool tail;                   // the last round of the second product may be split: its partial sums lie at off_tail behind y
    uint32_t few_splits;
    // ring1, ring2: rows of a tile of gemm_ring_kernel in the first and second product, 0: the kernels that tiled and m_tile name
    uint32_t m_tile, ksplit, ksplit1, split_tiles, ring1, ring2, pairs_cap, tiles_cap, n_chunks;
    uint64_t bytes;
    uint64_t off_count, off_offset, off_sorted, off_pos, off_tile, off_ntiles, off_h, off_y, off_part, off_tail;
};

inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// Shapes and launch parameters the FFN plan depends on (a routed layer, or one always-mapped expert
// for the shared-expert call).
struct FfnShape {
    uint64_t E, H, F;
    int n_cus, tiled_waves;
    bool ragged = false;         // the 256 x 256 tiles may be taken where H or F is not a multiple of 64
    bool routed = true;          // false: the shared expert, whose call has neither the kernels for few pairs nor a split last round
};

// k rows of a wavefront of gemm2_few_kernel: a quarter of its workgroup's, in whole MFMA steps
constexpr uint64_t kFewChunk = 32;
inline uint64_t few_quarter(uint64_t F, uint64_t splits) { return align_up((align_up((F + splits - 1) / splits, kFewChunk) + 3) / 4, kFewChunk); }

// First product in weight strips with K split k ways, in k rows of a workgroup (about 30 ns each when the memory system is not
// saturated): rounds of one workgroup per CU, each with a start-up of 128 rows; the launch that adds up the partial sums costs as much again,
// and their bytes, written and read, a row of a workgroup per KiB and CU.  kNoSplits where the rows do not make k splits of whole units.  cols:
// column workgroups, halves: the two pairs of wavefronts share the rows.
constexpr uint32_t kStripSplits = 16;
constexpr uint64_t kNoSplits = ~0ull;
inline uint64_t strip_cost(uint64_t H, uint64_t n_cus, uint64_t cols, uint64_t n_tiles, bool halves, uint64_t partial_bytes, uint64_t k) {
    if (k > 1 && k * 256 > H) return kNoSplits;
    const uint64_t unit = halves ? 256 : 128, k_per = align_up((H + k - 1) / k, unit);      // the kernel splits at multiples of that
    if (k > 1 && (H + k_per - 1) / k_per != k) return kNoSplits;
    const uint64_t rounds = (cols * n_tiles * k + n_cus - 1) / n_cus;
    return rounds * (std::min(k_per, H) / (halves ? 2 : 1) + 128) + (k > 1 ? 128 + k * partial_bytes / (n_cus * 1024) : 0);
}

// The few pairs' part of the plan p, which holds the general kernels' K splits, as many of them as fit `limit`: no sum is longer than
// with those, and what is chosen fits as well.  split: K splits of the first product are allowed; the general rule's would be splits_any
// in a buffer of any size.
inline void plan_few(FfnPlan& p, const FfnShape& c, uint32_t T, uint32_t K, uint64_t act, uint64_t pairs_act, bool split, bool halves_too,
                     uint32_t splits_any, uint64_t limit) {
    const uint64_t H = c.H, F = c.F, pairs = p.pairs_cap, n_cus = uint64_t(std::max(c.n_cus, 1));
    const uint64_t strips1 = (F + 127) / 128, strips2 = (H + 127) / 128;
    const uint64_t room = limit > p.off_y ? limit - p.off_y : 0;
    const auto sums1 = [&](uint64_t k) { return k > 1 ? align_up(k * pairs * 2 * F * 4, 256) : 0; };
    const auto sums2 = [&](uint64_t k) { return align_up(k * pairs * H * 4, 256); };
    // experts that T tokens of K distinct ones each are expected to touch
    double touched = std::max(1.0, double(act) * (1.0 - std::pow(1.0 - std::min(1.0, double(K) / double(c.E)), double(T))));
    // (a call that touches more of them than expected would take another round)
    if (T > 1 || act < c.E) touched = std::min({touched + 0.4 * std::sqrt(touched * (1.0 - touched / double(act))), double(act), double(pairs)});
    const uint64_t tiles = uint64_t(touched + 0.5);
    if (split && (strips1 + 1) / 2 * tiles < n_cus) {
        // The first product with the experts the call is expected to touch for its row tiles, and whole strips where they are as good (their
        // rows of weights are 512 bytes of a matrix, not 256).  Microseconds a call, general rule / here:
        // 160 experts of H 5120 F 1536, top-8, 4 tokens 242 / 228, 64 of H 2048 F 512, 17 tokens, top-2 44.6 / 41.6, 160 of H 5120
        // F 1536, 2 tokens, top-2 54 / 45, 64 of H 3000 F 136, 9 tokens, top-4 36.5 / 31.  Where whole strips are a round of workgroups already, the
        // general rule stays: other splits or halves then gain nothing that the estimate could see.  32 of H 1080 F 6360, 5 tokens, top-8 166 / 186, 64 of
        // H 2560 F 2176, 10, top-4 166 / 180, 42 of H 2960 F 9336, 10, top-4 809 / 882, 32 of H 3480 F 3200, 6, top-10 337 / 351.
        const auto chain = [&](uint64_t k, bool halves) { return std::min(H, align_up((H + k - 1) / k, halves ? 256 : 128)) / (halves ? 2 : 1); };
        // (as short as in a buffer that holds all of the general rule's splits, if something that is fits)
        for (const uint64_t longest : {chain(splits_any, p.halves), chain(p.ksplit1, p.halves)}) {
            uint64_t least[2] = {kNoSplits, kNoSplits};
            uint32_t best[2] = {0, 0};
            for (uint32_t k = 1; k <= kStripSplits; ++k)
                for (const bool halves : {false, true}) {
                    if ((halves && !halves_too) || chain(k, halves) > longest || sums1(k) > room) continue;
                    const uint64_t cost = strip_cost(H, n_cus, halves ? strips1 : (strips1 + 1) / 2, tiles, halves, pairs_act * 2 * F * 8, k);
                    if (cost < least[halves]) { least[halves] = cost; best[halves] = k; }
                }
            if (best[0] == 0 && best[1] == 0) continue;
            p.halves = best[1] && (best[0] == 0 || least[1] + least[1] / 64 < least[0]);
            p.ksplit1 = best[p.halves];
            break;
        }
    }
    // The second product in gemm2_few_kernel while its workgroups make one round, a wavefront's quarter of K is short and no longer than the sums
    // of gemm2_kernel, which is the faster one past either line.  Microseconds a call, gemm2_kernel / gemm2_few_kernel: 8 experts of H 2232,
    // 9 tokens, top-5 (144 workgroups), F 432 39.9 / 32.1, 864 (quarters of 224 k; gemm2_kernel sums 288) 41.0 / 38.8, 1024 (256; 256)
    // 39.7 / 39.5, but 1280 (320; 256) 42.3 / 43.4, 1728 (448; 288) 50.1 / 51.8; with three splits, 432 workgroups, the last two 45.2 and
    // 52.6; 160 of H 5120 F 384, 2 tokens, top-8 (640 workgroups) 42.4 / 45.6.  4 of H 4752 F 1680, 4 rows of each (quarters of 448 k against 288 k) 51.3 / 54.0, 15 rows 58.1 / 65.8.  One of H 4096 F 14336, one token
    // (256 workgroups, 448 k) 83 / 66, two (896 k) 122 / 119, but four (1792 k) 218 / 220.
    // Tiles of more than 16 rows take the body for 64, which is slower than gemm2_kernel: not where they are likely, with even routing or where
    // the most popular expert gets 0.3 of the tokens for each of their experts (16 experts by rank^-1.1).  Two of 4 experts a token, H 512 F 256, 26 tokens 24.5 / 26.6,
    // H 4736 F 512, 28 tokens 33.2 / 35.3; of 16 of H 2048 F 1024, 28 tokens by rank 39.7 / 44.4 (even 47.5 / 45.3), F 512, 32 tokens 32.5 / 36.4 (33.9 / 33.2); one of 8 of H 880
    // F 1960, 42 tokens 36.9 / 34.4; 15 tokens with four of 4, H 4192 F 232 36.5 / 32.
    const double rows_mean = double(pairs) / double(c.E), rows_most = rows_mean + 1.5 * std::sqrt(rows_mean * (1.0 - std::min(1.0, double(K) / double(c.E))));
    const bool short_tiles = T <= 16 || std::max(rows_most, double(T) * std::min(1.0, 0.3 * double(K))) <= 16.0;
    const uint64_t wgs = strips2 * tiles, longest = std::min(F, align_up((F + p.ksplit - 1) / p.ksplit, kFewChunk));
    const auto splits_in = [&](uint64_t free, uint64_t most_wgs, uint64_t most_rows) {      // 0: there are none
        uint64_t least = ~0ull;
        uint32_t best = 0;
        for (uint64_t k = 1; k <= 8 && (k == 1 || (k * 256 <= F && (split || k <= p.ksplit))); ++k) {
            const uint64_t rows = few_quarter(F, k);
            if (std::min(F, rows) > longest || rows > most_rows || wgs * k > most_wgs || sums2(k) > free) continue;
            const uint64_t rounds = (wgs * k + n_cus - 1) / n_cus, cost = rounds * (rows + 96) + (k > 1 ? 32 * k : 0);
            if (cost < least) { least = cost; best = uint32_t(k); }
        }
        return best;
    };
    // Fused where a quarter is at most 256 k in one round, 128 in a round and a half.  Microseconds a call, apart / fused: one token's top-10
    // of 512 of H 2048 F 512 26.0 / 24.3, of 64 of H 2048 F 640 28.6 / 27.4, F 1024 35.7 / 34.9, top-4 of H 4096 F 640 27.7 / 28.0, F 1024
    // 32.8 / 29.1, top-6 of H 5120 F 768 37.2 / 37.4, 4 tokens, top-4 of H 512 F 1024 20.8 / 20.9; three tokens, top-8 (F 256, 384
    // workgroups) 27.2 / 26.3; but one token's top-8 of H 5120 (320 workgroups) F 768 43.5 / 45.3; 16 tokens' rows cost more than the launch
    // (48.6 / 50.9).
    const bool one_round = wgs <= n_cus;
    if (split && p.ksplit1 > 1 && T <= 4 && few_quarter(F, 1) <= (one_round ? 256 : 128) && sums1(p.ksplit1) + sums2(p.ksplit) <= room)
        p.few_splits = splits_in(room - sums1(p.ksplit1), one_round ? n_cus : 3 * n_cus / 2, 256);
    p.few_fused = p.few_splits != 0;
    // (without room for gemm2_kernel's splits there is no call)
    if (!p.few_fused && short_tiles) p.few_splits = splits_in(std::max(room, sums2(p.ksplit)), n_cus, tiles <= 2 ? 1024 : 512);
}

// split: with K splits of the first product and 128 x 128 tiles; without them the plan takes the least scratch.
inline FfnPlan plan_ffn_rules(const FfnShape& c, uint32_t T, uint32_t K, uint32_t mapped, bool split, uint64_t limit) {
    FfnPlan p{};
    const uint64_t E = c.E, H = c.H, F = c.F;
    const uint64_t pairs = uint64_t(T) * K;
    const uint64_t groups = std::max<uint64_t>(1, std::min<uint64_t>(E, pairs));
    const uint64_t avg = (pairs + groups - 1) / groups;
    const uint64_t n_cus = uint64_t(std::max(c.n_cus, 1));
    // what a call with only `mapped` experts resident multiplies
    const uint64_t act = mapped ? std::min<uint64_t>(mapped, E) : E;
    const uint64_t pairs_act = std::max<uint64_t>(1, pairs * act / E);
    const uint64_t groups_act = std::max<uint64_t>(1, std::min(act, pairs_act));
    // Row tile of the weight-streaming kernels: every extra tile of an expert streams that expert's
    // weights again, and routing can be far from even, so tiles hold up to 128 rows (the kernel takes a
    // cheaper body for tiles with fewer rows).  With so many rows per expert that even 128-row tiles are
    // exceeded often (an expert's row count taken as normal with mean and variance avg), 128-row tiles
    // stay the choice while the expected number of passes per expert is below 1.6 - what one pass of
    // the LDS-tiled MFMA kernels (256-row tiles, k extents that are multiples of 64) costs relative to
    // a streaming pass at these sizes.
    auto p_over = [&](double m) { return 0.5 * std::erfc((m + 0.5 - double(avg)) / std::sqrt(2.0 * double(avg))); };
    const bool tileable = H % 64 == 0 && F % 64 == 0;
    // (their byte offsets into 256 rows of h have 32 bits)
    const bool tiles256 = F < (1u << 23) && (tileable || (split && c.ragged && c.tiled_waves == 2));
    p.m_tile = 128;
    if (p_over(128) > 0.02 && 1.0 + p_over(128) + p_over(256) + p_over(384) > 1.6 && tiles256)
        p.m_tile = 256;
    bool forced = false;
    if (const char* v = std::getenv("FLUXMOE_FFN_MTILE")) {
        const int m = std::atoi(v);
        if (m == 16 || m == 32 || m == 64 || m == 96 || m == 128 || (m == 256 && tileable && tiles256)) { p.m_tile = uint32_t(m); forced = true; }
    }
    p.tiled = p.m_tile == 256;
    // H or F that is not a multiple of 64: the 256 x 256 tiles take a partial step, so the same line holds.  Microseconds a call, 128-row strips /
    // tiles: 8 experts of H 3000 F 7000, 250 rows each 571 / 435, 1024 rows 1720 / 1208; 160 of H 2600 F 1000, 150 rows 1294 / 752; with the
    // splits that stand for the strips' halves (chains below) 64 of H 2000 F 312, 1250 rows 1089 / 905; one of H 5000 F 1496, 2000 rows 198 / 173.
    // Where the launch would leave CUs without a workgroup.  All figures: microseconds per call, weights out of HBM.
    if (split && !forced && tiles256 && c.tiled_waves == 2) {
        const double avg_act = double(pairs_act) / double(groups_act);
        const bool few_strips = 2 * ((F + 255) / 256) * groups_act <= n_cus;       // strip workgroups before any K split
        if (p.tiled) {
            // A single expert in 256 x 256 tiles: tiles of 128 x 128, two workgroups per CU, while the large ones fill three
            // quarters of the CUs at most.  H 5120 F 1536, tiles of 256 / 128: 512 rows (24 large tiles) 70 / 67, 2048 (96)
            // 157 / 144, 4096 (192) 262 / 235, 16384 792 / 921; H 2048 F 512: 256 rows 46 / 29, 2048 65 / 48.  H 4096 F 1792,
            // 4096 rows (224): 194 / 220; H 4096 F 4096, 2048 rows (256): 199 / 225.  Up to 512 rows the weights' way out of HBM
            // bounds the call and two workgroups keep more loads in flight, up to a round and a half: H 4096 F 14336, 512 rows
            // (224): 255 / 237.  Several experts with several row tiles each stay (20 of H 5120 F 1536, 205 rows: 383 / 451).
            // T rows, not the mean of what one of several experts gets: a batch may be routed to it alone.
            if (tileable && groups_act == 1 && (T <= 512 ? 2 : 4) * ((uint64_t(T) + 255) / 256) * ((F + 127) / 128) <= 3 * n_cus) p.m_tile = 128;
        } else if (few_strips && groups_act > 1 && 0.5 * std::erfc((128.5 - avg_act) / std::sqrt(2.0 * avg_act)) > 0.02) {
            // Experts that often need a second 128-row strip tile: 8 of H 4096 F 1792, 128 rows each: strips 172, tiles of 256 121.
            p.tiled = true;
            p.m_tile = 256;
        } else if (tileable && few_strips && (groups_act == 1 ? pairs_act >= 64 && H * F * 6 <= (64u << 20)
                                                  : 8 * groups_act <= n_cus && avg_act >= 16 && H <= (mapped && mapped < E ? 2048u : 1024u))) {
            // Row counts that make a matrix tile worth while and K too short for the strips' start-up, strips / tiles of 128:
            // one expert, weights out of HBM and behind a kernel that filled the caches with other data: H 2048 F 512, 64 rows
            // 30 / 26 and 36 / 35, 128 44 / 27 and 52 / 37; H 5120 F 1536, 64 rows 45 / 45 and 48 / 57, 96 54 / 48 and 57 / 59,
            // 128 63 / 51 and 66 / 63.  Past 64 MiB of weights they gain in the one state what they lose in the other: H 4096
            // F 4096, 96 rows 63 / 61 and 68 / 81, F 14336 115 / 146 and 120 / 190.  32 experts of H 1024 F 256, 40 rows each:
            // 39 / 36 and 46 / 48, 87 rows 59 / 40 and 65 / 52; of H 2048 F 512, 16 rows each: 55 / 58 and 62 / 93, and 64 of
            // those, 20 rows: 85 / 106 and 91 / 154.  A wave (part of the layer resident) runs beside the next wave's load, and
            // there they win, likely because a strip workgroup needs 128 KiB of LDS on a CU that decodes and a tile 80: a pass
            // over three layers of 128 of H 2048 F 512 in waves of 32, 1024 tokens: 2217 / 2040; in waves of 64 they lose
            // (1620 / 1690).
            // Longer K favours the strips: 20 of H 5120 F 384, 51 rows each: 79 / 99; 8 of H 4096 F 1792, 64 rows: 101 / 109.
            p.tiled = true;
            p.m_tile = 128;
        }
    }
    p.pairs_cap = uint32_t(std::max<uint64_t>(pairs, 1));
    p.tiles_cap = uint32_t(pairs / p.m_tile + groups + 1);
    // Split K of the second product (strip kernels).  One workgroup (four strips, one per SIMD) fits on a
    // CU at a time, so the launch runs in rounds of n_cus workgroups; the split is the one with the
    // smallest estimated time in units of k rows per workgroup: rounds x (rows per split + a fixed
    // start-up cost) + the FP32 partials it writes and combine_kernel reads back.
    const uint64_t strips2 = (H + 127) / 128;
    const uint64_t est_tiles = std::max<uint64_t>(1, std::max<uint64_t>(pairs / p.m_tile, std::min(groups, pairs)));
    uint64_t ks = 1, best_cost = ~0ull;
    for (uint64_t k = 1; k <= 8 && k <= std::max<uint64_t>(1, F / 256); ++k) {
        const uint64_t wgs = (strips2 + 3) / 4 * est_tiles * k;
        const uint64_t rounds = (wgs + n_cus - 1) / n_cus;
        const uint64_t partials = k > 1 ? k * pairs * H * 8 / (n_cus * 1024) : 0;
        const uint64_t cost = rounds * ((F + k - 1) / k + 384) + partials;
        if (cost < best_cost) { best_cost = cost; ks = k; }
    }
    p.ksplit = uint32_t(ks);
    p.ksplit1 = 1;
    // Tiles where H or F is no multiple of 64 stand in for strips, and a sum of either product is as long as it would be there at
    // most: the strips' K splits and halves are kept as splits (8 experts of H 4400 F 3504, 140 rows each: share of tokens with
    // an h rounded the other way 0.225 in strips' halves, 0.271 unsplit).
    uint32_t chains = 1, chains2 = 1;
    if (p.tiled && !tileable) {
        FfnShape strips = c;
        strips.ragged = false;
        const FfnPlan q = plan_ffn_rules(strips, T, K, mapped, split, limit);
        chains = q.ksplit1 * (q.halves ? 2u : 1u);
        chains2 = q.ksplit;
        // Short K: the partial sums cost more than the tiles gain, the more so where the memory-side cache (256 MB) does not hold
        // them.  Microseconds, strips / two splits: within it 8 experts of H 528 F 2632, 182 rows each 81 / 90, H 816 F 1016, 309 rows
        // 78 / 68, H 928 F 392, 881 rows 83 / 72; past it H 608 F 896, 9395 rows 748 / 808, 160 of H 728 F 272, 498 rows 480 / 499,
        // of H 1224 F 896, 134 rows 533 / 493, of H 2496 F 1400, 391 rows 3091 / 2583.
        if (chains > 1 && H < (chains * pairs_act * 2 * F * 4 > (256u << 20) ? 512u : 384u) * chains) return q;
        p.ksplit1 = chains;
    }
    p.few = c.routed && !p.tiled && p.m_tile >= kFewPairs && pairs <= kFewPairs;
    // LDS-tiled kernels: row tiles to expect, and nanoseconds a product of `tiles` tiles and `steps` steps of 64 k takes when
    // split k ways.  A tile costs 3 us to start; a step 1.4 us (256 x 256, one workgroup per CU), or 0.56 us (128 x 128)
    // alone on a CU and 0.88 us for each of two.  Partial sums are written and read at 10 TB/s (mostly in the caches).
    const uint64_t row_tiles = groups_act == 1 ? (pairs_act + p.m_tile - 1) / p.m_tile
                                               : std::max(groups_act, pairs_act / p.m_tile + groups_act / 2);
    auto tile_ns = [&](uint64_t tiles, uint64_t steps, uint64_t k) {
        const uint64_t wgs = tiles * k, per = (steps + k - 1) / k;
        if (p.m_tile == 256) return (wgs + n_cus - 1) / n_cus * (per * 1400 + 3000);
        const uint64_t full = wgs / (2 * n_cus), rest = wgs % (2 * n_cus);
        return full * (per * 880 + 3000) + (rest == 0 ? 0 : per * (rest <= n_cus ? 560 : 880) + 3000);
    };
    if (p.tiled) {
        // When the second product has fewer tiles than the chip has CUs, the LDS-direct kernels split K so that about one
        // workgroup per CU runs (each split keeps at least 8 steps of 64)
        p.ksplit = 1;
        if (p.m_tile == 128) {
            uint64_t best = ~0ull;
            for (uint64_t k = 1; k <= 8 && (k == 1 || (k * 512 <= F && row_tiles * ((H + 127) / 128) * k <= 2 * n_cus)); ++k) {
                const uint64_t cost = tile_ns(row_tiles * ((H + 127) / 128), F / 64, k) + k * pairs_act * H * 8 / 10000;
                if (cost < best) { best = cost; p.ksplit = uint32_t(k); }
            }
        } else if (c.tiled_waves == 2 || c.tiled_waves == 1) {
            const uint64_t tiles2 = groups * ((avg + 255) / 256) * ((H + 255) / 256);
            uint64_t k2 = std::max<uint64_t>(1, n_cus / tiles2);
            k2 = std::min<uint64_t>(k2, 8);
            k2 = std::min<uint64_t>(k2, std::max<uint64_t>(1, F / 512));
            p.ksplit = std::max(uint32_t(k2), chains2);
        }
    }
    // K split of the first product, for launches that would leave most of the chip without a workgroup: the FP32 partial
    // sums of gate and up cost a write, a read and a launch.  Measured, whole FFN call: one token, top-10 of 512 experts,
    // H 2048 F 512 (20 workgroups unsplit) 63 -> 36 us; 333 tokens, top-4 of 64, H 2880 F 360 (128) 140 -> 116 us.  Layers
    // whose tiles fill the chip stay unsplit (8 experts of H 4096 F 14336: 448 workgroups).
    if (split && (!p.tiled || c.tiled_waves == 2)) {
        const uint64_t partial_bytes = pairs_act * 2 * F * 8;             // written and read, per split
        uint64_t best = ~0ull;
        if (!p.tiled) {
            const uint64_t strips1 = (F + 127) / 128, tiles1 = std::max<uint64_t>(pairs_act / p.m_tile, groups_act);
            auto consider = [&](bool halves) {
                for (uint32_t k = 1; k <= kStripSplits; ++k) {
                    const uint64_t cost = strip_cost(H, n_cus, halves ? strips1 : (strips1 + 1) / 2, tiles1, halves, partial_bytes, k);
                    if (cost < best) { best = cost; p.ksplit1 = k; p.halves = halves; }
                }
            };
            consider(false);
            if (p.m_tile == 128 && !forced && (strips1 % 2 || (strips1 + 1) / 2 * tiles1 < n_cus)) consider(true);
        } else {
            const uint64_t cols = p.m_tile / 2;
            const uint64_t tiles1 = row_tiles * ((F + cols - 1) / cols), room = p.m_tile == 256 ? n_cus : 2 * n_cus;
            for (uint64_t k = chains; k <= std::max(8u, chains) && (k == chains || (k * 512 <= H && tiles1 * k <= room)); ++k) {
                const uint64_t cost = tile_ns(tiles1, H / 64, k) + (k > 1 ? 4500 + k * partial_bytes / 10000 : 0);
                if (cost < best) { best = cost; p.ksplit1 = uint32_t(k); }
            }
        }
    }
    // Strips whose rows are not whole 128-byte lines share a line with their neighbours: on one XCD they find it in its L2
    // (64 experts of H 2880 F 360, 333 tokens, top-4: 112 -> 107 us, 80 of F 376 127 -> 114, 64 of H 2048 F 200, 500 tokens
    // 66 -> 62, of H 1544 F 264, 600 tokens 71 -> 66; 160 of F 104, one strip each, 84 -> 85).  With aligned rows it changes nothing
    // (64 of F 384: 94.4 / 93.5), with two strips a workgroup it is 0.5 to 2 % slower.  Enough (tile, split) units to fill the
    // 8 XCDs evenly.
    p.g1_xcd = !p.few && p.halves && F % 64 != 0 && groups_act * p.ksplit1 >= 64;
    // The last round of the second product: tiles of 256 x 256, unsplit, long K, more than a round of them.
    p.tail = c.routed && split && p.tiled && p.m_tile == 256 && c.tiled_waves == 2 && p.ksplit == 1 && F >= kLastRoundF && row_tiles * ((H + 255) / 256) > n_cus;
    uint64_t o = 0;
    auto take = [&](uint64_t bytes) { uint64_t at = o; o = align_up(o + bytes, 256); return at; };
    p.off_count = take((E + 1) * 4);
    p.off_offset = take((E + 2) * 4);
    p.off_sorted = take(uint64_t(p.pairs_cap) * 4);
    p.off_pos = take(uint64_t(p.pairs_cap) * 4);
    p.off_tile = take(uint64_t(p.tiles_cap) * 16);
    p.off_ntiles = take(8);
    p.n_chunks = pairs > kRouteChunkThreshold ? uint32_t((pairs + kRouteChunkPairs - 1) / kRouteChunkPairs) : 0u;
    p.off_h = take(std::max<uint64_t>(uint64_t(p.pairs_cap) * F * 2, uint64_t(p.n_chunks) * E * 4));
    p.off_y = o;
    uint32_t general2 = 0;
    // the partial sums of the first product are read before the second product writes its own in the same place
    auto end = [&]() {
        // (with room for gemm2_kernel's splits also where gemm2_few_kernel takes fewer: a buffer without it was never enough)
        const uint64_t y = align_up(uint64_t(std::max(p.ksplit, general2)) * p.pairs_cap * H * 4, 256);
        const uint64_t part = p.ksplit1 > 1 ? align_up(uint64_t(p.ksplit1) * p.pairs_cap * 2 * F * 4, 256) : 0;
        p.off_part = p.few_fused ? p.off_y + y : p.off_y;
        const uint64_t sums = std::max(p.off_y + y, p.off_part + part);
        p.off_tail = sums;
        return p.tail ? sums + kTailBytes : sums;
    };
    if (p.tail && end() > limit) p.tail = false;
    const uint32_t splits_any = p.ksplit1;
    if (split)
        while (p.ksplit1 > chains && end() > limit) --p.ksplit1;
    if (p.few) {
        plan_few(p, c, T, K, act, pairs_act, split, p.m_tile == 128 && !forced, splits_any, limit);
        general2 = p.ksplit;
        if (p.few_splits) p.ksplit = p.few_splits;
    }
    if (split) {
        if (chains > 1) {
            p.split_tiles = ~0u;
        } else if (p.ksplit1 > 1 && p.tiled && p.m_tile == 256) {
            const SplitShape s{uint32_t(H), uint32_t(F), uint32_t(n_cus)};
            const auto cost = [&](uint32_t k) { return tiled_cost(s, uint32_t(row_tiles), uint32_t(pairs_act), k); };
            p.split_tiles = uint32_t(row_tiles);
            for (uint32_t k = 1; k < p.ksplit1; ++k) if (cost(k) <= cost(p.ksplit1)) p.split_tiles = 0;
        } else if (p.ksplit1 > 1) {
            const uint64_t cols = p.tiled ? (F + 63) / 64 : (p.halves ? (F + 127) / 128 : (F + 255) / 256);
            const uint64_t planned = p.tiled ? row_tiles : std::max<uint64_t>(pairs_act / p.m_tile, groups_act);
            p.split_tiles = uint32_t(std::max((n_cus - 1) / cols, planned));
        }
        while (p.tiled && p.m_tile == 128 && p.ksplit > 1 && end() > limit) --p.ksplit;
        while (p.tiled && !tileable && p.ksplit > chains2 && end() > limit) --p.ksplit;
    }
    p.bytes = end();
    return p;
}

// limit: bytes the scratch may take (the call's buffer; the size query leaves it open): the splits give way to it, then the
// tiles that stand in for strips do, whose halves need no partial sums, and then the small tiles, so a buffer that holds the plan
// without them is always enough.  The small tiles also give way where there would be too many of them.
// mapped: experts of the layer known to be resident, 0 = not known (it steers speed, not what is accepted).
inline FfnPlan plan_ffn(const FfnShape& c, uint32_t T, uint32_t K, uint64_t limit = ~0ull, uint32_t mapped = 0) {
    auto fits = [&](const FfnPlan& p) { return p.bytes <= limit && p.tiles_cap <= kMaxRowTiles; };
    const FfnPlan p = plan_ffn_rules(c, T, K, mapped, true, limit);
    if (fits(p)) return p;
    if (c.ragged && (c.H % 64 != 0 || c.F % 64 != 0)) {
        FfnShape strips = c;
        strips.ragged = false;
        const FfnPlan q = plan_ffn_rules(strips, T, K, mapped, true, limit);
        if (fits(q)) return q;
    }
    return plan_ffn_rules(c, T, K, mapped, false, limit);
}

// Scratch the size query asks for: enough for the plan a call prefers and for the one it falls back on.  The splits that tiles
// take in the strips' place only keep sums short, and strips halve theirs without any memory: no more than 64 MB are asked for
// them (8 experts of H 4400 F 3504, 140 rows each, within it 353 / 262 us; of H 1856 F 2632, 1646 rows each, past it: 167 MB, 624 with the
// splits).  A call whose buffer has the room takes them all the same.
inline uint64_t ffn_bytes(FfnShape c, uint32_t T, uint32_t K) {
    const FfnPlan p = plan_ffn_rules(c, T, K, 0, true, ~0ull);
    const uint64_t tiles = p.bytes - (p.tail ? kTailBytes : 0);
    c.ragged = false;
    uint64_t strips = std::max(plan_ffn_rules(c, T, K, 0, true, ~0ull).bytes, plan_ffn_rules(c, T, K, 0, false, ~0ull).bytes);
    // few pairs: with part of the layer resident there are fewer row tiles and more splits, the most with some number between
    // one and all of them (16 experts of H 2048 F 12728, 7 tokens, top-7: 4.5 MB with all, 21 with 6)
    if (p.few)
        for (uint32_t mapped = 1; mapped < c.E; ++mapped) strips = std::max(strips, plan_ffn_rules(c, T, K, mapped, true, ~0ull).bytes);
    return tiles <= strips + (64ull << 20) ? std::max(tiles + (p.tail ? kTailBytes : 0), strips) : strips;
}

// Whether combine_kernel reads the second product's partial sums (`bytes` for all T * K pairs) and writes the output with the
// non-temporal hint: for sums larger than the memory-side cache (256 MB), each of which is read once, while what it would push out is
// the sums still to be read.  Microseconds of the kernel, default policy / non-temporal: 234 MB 42 / 42, 312 MB 78 / 58, 390 MB 109 / 82,
// 640 MB 164 / 136 (H 5120, top-8), 937 MB 248 / 214 (H 2048, top-10).  A call with part of the layer resident has the sums of
// those experts only: 4096 tokens, 80, 40 of 160 experts of H 5120, top-8 (336, 168 MB) 80 / 78, 51 / 65; 256 of 512 of H 2048, top-10
// (168 MB) 39 / 45.
inline bool combine_streams(uint64_t bytes, uint64_t mapped, uint64_t E) {
    return (mapped && mapped < E ? bytes / E * mapped : bytes) > (256ull << 20);
}

// Whether the LDS-direct kernels fetch a layer's weights with the non-temporal hint.  Weights that one row tile reads (experts
// with about a tile's rows at most) pass the caches by; with several they are shared through L2.  Microseconds a call, default
// policy / non-temporal: 8 experts of H 4096 F 14336, 250 rows each 950 / 890, 1024 rows 2768 / 2807; 20 of H 5120 F 1536, 240 rows 377 / 361,
// 1200 rows 1207 / 1279; behind the load of the whole layer, load included, 1880 / 1774 and 693 / 676.
// A layer that the memory-side cache (256 MB) may hold from the call before is read from there: 32 of H 1024 F 256 (50 MB), 75 rows
// 32.7 / 36.6 (out of HBM 39.7 / 37.6); of H 2048 F 512 (201 MB), 200 rows, two layers in turn 118 / 110.
// With many experts skew gives some of them several tiles: 160 of H 5120 F 1536, even routing, 205 rows 2080 / 2062, popularity by
// rank, 175 rows 2270 / 2291; 512 of H 2048 F 512, 234 rows 1415 / 1438.  Waves find what their load just wrote: a pass over 128 of
// those 2012 / 2040.
inline bool weights_stream(uint64_t E, uint64_t H, uint64_t F, uint64_t pairs, uint64_t m_tile) {
    return E <= 64 && E * H * F * 6 > (128ull << 20) && pairs <= m_tile * std::min(E, pairs);
}

// Whether a walking launch of 256 x 256 tiles with n_ct column tiles takes them row by row and not in super-tiles.  group: super-rows
// in a group of super-tiles that were asked for, 0 for none.
// Experts of about one row tile share no weights between their tiles, and what is left to share are the activations: with few
// column tiles an XCD's 32 tiles are taken row by row, so that a row's columns run together (12 column tiles in super-tiles of 8 x 4
// fetched every row of activations three times) and no place stays empty.  Microseconds a call, super-tiles / rows: 160 experts
// of H 5120 F 1536, 205 rows each 2032 / 1992, 300 rows 3599 / 3491, 80 of them, popularity by rank, 137 rows 1046 / 1021; one to eight
// column tiles are the same order, or nearly: 512 of H 2048 F 512, 200 rows 1071 / 1067, 256 of them, 300 rows 1005 / 1011.  More rows:
// 400 to 450 of them still gain (160 of H 5120 F 1536, 450 rows 4069 / 3853), 512 do not (4536 / 4541; 31 of H 2048 F 5120 1104 / 1123), 20
// experts with 1392 rows 1369 / 1392.  More columns, up to 384 rows: what even routing gains (40 of H 2048 F 3200, 205 rows 458 / 435, 31 of F 5120
// 502 / 502, 22 of F 7168 543 / 512), popularity by rank loses (64 of F 4096, 187 rows 967 / 991, 8 of H 4096 F 3584, 300 rows 310 / 326).
inline bool tiles_by_rows(uint64_t n_ct, uint64_t avg_rows, uint32_t group) { return group == 0 && n_ct <= 24 && avg_rows <= 384; }

// One product of the shared expert in gemm_ring_kernel: rows of a tile and K splits with the least estimated time.
struct RingProduct {
    uint32_t rows, splits;
    uint64_t wgs, cap, ns;        // workgroups, how many run at a time, nanoseconds
};
// T rows, K x N matrix (first product: gate and up of N columns).  A workgroup takes 4.5 us to start and end and, per step of 64 k,
// 0.40, 0.49 or 0.60 us (tiles of 32, 64, 128 rows) alone on a CU and 0.65 or 0.80 us for each of two; no faster than weights
// leave HBM at 5.4 TB/s.  Splits cost a launch and their partial sums at 10 TB/s.  Measured, one product, weights out of HBM, without the
// launch (model): H 5120 F 1536, first, 512 rows: 128 rows unsplit 50 (53), two splits 36 (36), 64 rows 42 (44), four splits 42;
// second, 128 rows 20 (19), 64 rows 21 (24), 32 rows 27.
inline RingProduct ring_product(uint64_t n_cus, uint64_t T, uint64_t K, uint64_t N, bool first) {
    RingProduct best{0, 0, 0, 0, ~0ull};
    const uint64_t steps = (K + 63) / 64, col_tiles = first ? (N + 63) / 64 : (N + 127) / 128;
    const uint64_t bytes = K * N * (first ? 4 : 2), out_bytes = T * N * (first ? 16 : 8);     // of a split, written and read
    for (const uint64_t rows : {32u, 64u, 128u}) {
        const uint64_t alone = rows == 32 ? 400 : (rows == 64 ? 490 : 600), paired = rows == 32 ? 650 : 800;
        const uint64_t cap = rows == 128 ? n_cus : 2 * n_cus, tiles = (T + rows - 1) / rows * col_tiles;
        for (uint64_t k = 1; k <= 8 && (k == 1 || (2 * k <= steps && tiles * k <= cap)); ++k) {
            const uint64_t per = (steps + k - 1) / k, wgs = tiles * k, rest = wgs % cap;
            uint64_t ns = wgs / cap * (per * (rows == 128 ? alone : paired) + 4500);
            if (rest) ns += per * (rest <= n_cus ? alone : paired) + 4500;
            ns = std::max(ns, bytes * 10 / 54 / 1000 + 4500) + (k > 1 ? 4500 + k * out_bytes / 10000 : 0);
            if (ns < best.ns) best = RingProduct{uint32_t(rows), uint32_t(k), wgs, cap, ns};
        }
    }
    return best;
}

// The shared expert (every token once on one dense expert).  While the first product fits one round of workgroups and the second two,
// both run in gemm_ring_kernel, which takes any H and F and lets the second product write the output itself where it is not
// split.  Microseconds a call, weights out of HBM, other kernels / ring: H 5120 F 1536, 1 row 31 / 23, 64 rows 46 / 28, 512 rows 67 / 58;
// H 2048 F 512, 211 rows 31 / 18, 1024 rows 40 / 27; H 4096 F 14336, 3 rows 88 / 70, 128 rows 128 / 93; H 4504 F 2776, 241 rows
// 126 / 71, 700 rows 210 / 189; H 1000 F 200, 50 rows 35 / 15.
// Where H and F are whole steps the other LDS-direct kernels win with two workgroups on a CU in the first product or two long
// rounds in the second: H 5120 F 1536, 1344 rows 116 / 136, 1024 rows 91 / 97, 2048 rows 134 / 170; but H 5120 F 384, 1024 rows 48 / 41.
inline FfnPlan plan_shared(FfnShape c, uint32_t T, uint64_t limit = ~0ull) {
    c.routed = false;
    const FfnPlan base = plan_ffn(c, T, 1, limit);
    const uint64_t n_cus = uint64_t(std::max(c.n_cus, 1));
    const RingProduct first = ring_product(n_cus, T, c.H, c.F, true), second = ring_product(n_cus, T, c.F, c.H, false);
    if (c.tiled_waves != 2 || std::getenv("FLUXMOE_FFN_MTILE") || first.wgs > first.cap || second.wgs > 2 * second.cap) return base;
    if (c.H % 64 == 0 && c.F % 64 == 0 && (first.wgs > first.splits * n_cus || (second.wgs > second.cap && c.F >= 1024))) return base;
    FfnPlan p = base;
    p.tiled = p.halves = p.g1_xcd = false;
    p.ring1 = first.rows;
    p.ring2 = second.rows;
    p.ksplit1 = first.splits;
    p.ksplit = second.splits;
    // the two products' partial sums lie in the same place: where the buffer is short, the larger of them gives way
    for (;;) {
        const uint64_t y = p.ksplit > 1 ? uint64_t(p.ksplit) * T * c.H * 4 : 0, part = p.ksplit1 > 1 ? uint64_t(p.ksplit1) * T * 2 * c.F * 4 : 0;
        p.bytes = p.off_y + align_up(std::max(y, part), 256);
        if (p.bytes <= limit) return p;
        if (y == 0 && part == 0) return base;
        if (part >= y) --p.ksplit1; else --p.ksplit;
    }
}

inline uint64_t shared_bytes(FfnShape c, uint32_t T) {
    c.routed = false;
    const uint64_t base = ffn_bytes(c, T, 1);
    c.ragged = false;
    return std::max(base, plan_shared(c, T).bytes);
}

}  // namespace fluxmoe
