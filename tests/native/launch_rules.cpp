// The launchers' rules as C functions, for tests without a GPU.
#include "launch_rules.h"

using namespace heatkv;

extern "C" int calibration_f32_per_unit(int d, int n_scales, unsigned blocks, int fit) {
  return rules::calibration_f32_per_unit(d, n_scales, blocks, fit);
}

extern "C" int copying_wavefronts(int d, unsigned attend_blocks, unsigned copy_blocks, unsigned tiles) {
  return rules::copying_wavefronts(d, attend_blocks, copy_blocks, tiles);
}

extern "C" int two_key_streams(int d, unsigned attend_blocks, unsigned update_blocks, unsigned tiles) {
  return rules::two_key_streams(d, attend_blocks, update_blocks, tiles);
}
