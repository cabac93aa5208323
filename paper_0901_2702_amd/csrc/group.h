// Kernel argument block and launch helpers of the group inverter (group.hip): a
// wave per pixel pass.  routes.h says which launches it is for.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace vfisv {

// The synthesis points of an instrument in chunks of GROUP_PTS, one per lane
// (the tables end with a whole chunk; padding points repeat the last one and
// have no taps), and their taps.
constexpr int GROUP_PTS = 64;
struct GroupTables {
  const float* dl = nullptr;    // [n_chunk * GROUP_PTS] offsets, in record order (dense: 1 chunk)
  const float* taps = nullptr;  // dense: [6][GROUP_PTS], natural row order; banded: [n_obs][16]
                                // over the row's 4 blocks
  int n_chunk = 0;
};

struct GroupArgs {
  LMArgs A;
  GroupTables T;
  long long n_max;  // pixels up to which this kernel serves the launch; a launch whose
                    // count is only known on the device exits at once above it
};
// work[] slot (behind the counters) where a launch over a device-side count
// leaves the pixels it did not serve: all of them or none.
constexpr int GROUP_LEFT_SLOT = QUEUE_SLOT0 - 1;
static_assert(GROUP_LEFT_SLOT >= COUNTER_SLOTS, "a slot of its own");

// Most pixels a wave works on at a time, per layout (KIND_*): as many as leave
// room for eight waves' LDS on a CU, two per SIMD.
constexpr int GROUP_SLOTS[2] = {8, 8};

// Synthesis by waves of a few models; num_cus sizes the grid.
hipError_t launch_synth_group(const SynthArgs& a, const GroupTables& t, int kind, bool deriv,
                              int num_cus, hipStream_t s);
hipError_t launch_lm_group(const GroupArgs& a, int kind, int grid, hipStream_t s);
hipError_t lm_group_blocks_per_cu(int kind, int* out);

}  // namespace vfisv
