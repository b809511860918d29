// Launch shape of the decode kernel.  Host arithmetic only, without HIP, so that the rule can be tested on its own.
#pragma once

#include <algorithm>
#include <cstdint>

namespace fluxmoe {

// Blocks of a workgroup of `waves` wavefronts in a launch of `total` blocks; asked: blocks of a wavefront, 0 for the rule's choice.  Fewer
// than asked for where that would leave CUs without a workgroup.
// Up to 1536 blocks per CU a wavefront takes one block: a workgroup's life is then as short as it can be, and that is what a launch's
// ramp-up and its end cost.  Up to three blocks / one, microseconds a load, experts of 6 MB: 20 of them 44.7 / 40.6, 64 (69000 blocks) 135.5 / 132.0,
// 145 293.5 / 287.7, 200 (217000) 396 / 389; of 47 MB: 4 62.7 / 57.5, 20 on two streams 297 / 286, 40 (325000) 556 / 550.  Beyond it is even or
// worse: 60 of 47 MB (488000) 849 / 855, 8 of 352 MB (486000) 828 / 824, and with its FFN in turn 1321 / 1327, where 40 of 47 MB have
// 933 / 931 and 145 of 6 MB 500 / 498.  Passes of waves of 139000 blocks 1651 / 1642, 163000 2910 / 2880, 325000 3699 / 3695.
// Workgroups of four wavefronts with one block are faster alone (8 of 352 MB 811), but not before or beside an FFN (in turn 1331; a pass with
// waves of 35000 blocks 2042 / 2025 / 2062).
inline uint64_t decode_per_workgroup(uint64_t total, uint64_t n_cus, uint64_t waves, uint64_t asked) {
    const uint64_t per_wave = asked ? asked : (total <= 1536 * n_cus ? 1 : 3);
    return std::max(waves, std::min(waves * per_wave, total / (3 * n_cus)));
}

}  // namespace fluxmoe
