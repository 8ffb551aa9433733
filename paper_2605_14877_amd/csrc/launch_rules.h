// Rules of the launchers that follow from sizes alone: host code without HIP, so that both sides of a line can be checked
// without a GPU.
#pragma once

namespace heatkv {
namespace rules {

// Workgroups of calibrate_f32_kernel that may share a compute unit: the registers allow seven at d = 64 and four at d = 128,
// the LDS (`fit`) as many up to 10 and 15 scales.
// One scale, d = 128: three or four, whichever needs fewer turns times workgroups side by side; three where neither does.  Three
// -> four: 32 pairs, 400 x 921 keys (800 workgroups) 50 -> 45 us, 64 pairs 256 x 521 (1024) 41 -> 32 and 400 x 921 (1600) 80 -> 74, 256
// pairs 64 x 121 (1024) 23 -> 17; but 256 pairs 144 x 265 (2304) 46.5 -> 49, 32 and 64 pairs 144 x 265 (288, 576) 14.2 -> 14.6 and
// 18.1 -> 18.6.
// One scale in a turn of all that fit and a bit: two even turns of fewer.  d = 128 where four do not fit, three -> two: 64 pairs,
// 225 x 1310 (960) 88.5 -> 77.4, 80 pairs, 169 x 889 (880) 66.4 -> 59.6, 104 pairs, 144 x 720 (936) 57.6 -> 52.0; with four that do
// fit 784 and 800 are 1 to 2 % slower so.  d = 64, seven -> six: 64 pairs, 491 x 1470 (1984) 76.9 -> 70.9, 48 pairs, 635 x 1156 (1920)
// 60.8 -> 56.3; 1840 the same, 2064 and more 0 to 1 % slower.
// Several scales: the workgroups of the largest come first and take longest, so turns say nothing.  d = 128: a unit with four of
// them is done late, unless there are short ones enough to fill the others meanwhile: more than a turn of four and one of three
// take.  All scales in one call, three -> four: 16 pairs, up to 400 rows (960 workgroups) 34.7 -> 35.4, 40 pairs, up to 276 (1720)
// 46.7 -> 50.5 (but seven scales of 20 to 80 rows, 1000, 24.2 -> 22.3); 80 pairs, 20 to 80 (2000) 39.6 -> 36.8, 104 pairs, up to 276
// (4472) 103 -> 93.2, 512 pairs, up to 243 (13312) 217 -> 193.  d = 64, four -> seven: 40 pairs, up to 276 (1720) 32.7 -> 26.7; nothing
// that was timed loses.
inline int calibration_f32_per_unit(int d, int n_scales, unsigned blocks, int fit) {
  if (d == 64) return n_scales == 1 && blocks > 1824 && blocks <= 2048 && fit > 6 ? 6 : fit;
  const bool four = n_scales > 1 ? blocks > (4 + 3) * 256 : (blocks + 767) / 768 * 3 > (blocks + 1023) / 1024 * 4;
  if (four && fit >= 4) return 4;
  return n_scales == 1 && blocks > 800 && blocks <= 1024 ? 2 : 3;
}

}  // namespace rules
}  // namespace heatkv
