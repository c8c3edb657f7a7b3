// lbmd_tag.h -- the tags of the resident sub-cycle's exchange (no HIP needed).
#pragma once
#include <stdint.h>

namespace lbmd {

// A pass of a cycle publishes into slots that the pass before it, and the cycle
// before, used as well, and nothing empties them: a value that a segment left
// there after another had given its pass up may not pass for one of the next.
// So the tag of stage s of pass p of cycle n is (2^32 (2 n + p) + s) TAG, one
// value per stage of every pass (TAG is odd).
constexpr uint64_t RES_TAG = 0x9E3779B97F4A7C15ull;
constexpr uint64_t res_tag(uint64_t cycle, uint32_t pass, uint32_t stage) {
  return (((2 * cycle + pass) << 32) + stage) * RES_TAG;
}

}  // namespace lbmd
