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

// bf16 attention, launches of at most 256 workgroups that take a compute unit each, also those that copy rows of the cache
// update: do these find free units, or units that short walks leave, before the longest walk (`tiles` of 64 keys) is over?
// `attend_blocks`: workgroups that have queries (the grid is padded to a multiple of 8 pairs, those without end at once).
// Fitted, like the lines below, to 1200 launches of two-stream shapes at d = 64 and 2600 each of others, with bf16 and 8-bit rows.
inline bool update_finds_units(int d, unsigned attend_blocks, unsigned update_blocks, unsigned tiles) {
  return update_blocks <= 9 * (256 - attend_blocks) / 2 + (d == 64 ? 14 : 22) * tiles;
}

// Wavefronts that only copy tiles, on the SIMDs of those that compute, where a workgroup has one key stream.  One launch,
// without -> with them: d = 128, 48 pairs, 196 tokens 13.9 -> 13.1 us, 324 19.2 -> 17.8; 64 pairs, 144 10.2 -> 9.7; 128 pairs, 256
// (256 workgroups) 15.8 -> 14.8; d = 64, 64 pairs, 196 10.9 -> 10.3, 324 14.7 -> 13.9.  8-bit cache rows, where all eight
// wavefronts convert: a 2B-like layer, 13 scales, batch 1 611 -> 574, batch 2 828 -> 802; 12 heads, batch 3, up to 361 tokens 264
// -> 241.  Not for walks of one tile, which have nothing to copy ahead (8-bit rows 4.27 -> 4.37), nor where the update's
// workgroups would wait for units.  Two lines, workgroups of attention + update, tiles of the longest walk: for short walks d =
// 128, 96 + 192, 4 9.4 -> 9.0; 128 + 256, 4 10.2 -> 10.4; 192 + 270, 10 15.8 -> 15.1; 256 + 360, 10 17.1 -> 19.4; 256 + 512, 4 15.7 ->
// 19.2; for long ones the line above, 8-bit rows, 256 + 208, 10 19.4 -> 17.4; 256 + 378, 20 32.3 -> 28.0; 200 + 480, 23 36.2 -> 31.7;
// but 256 + 320, 14 23.2 -> 24.7; 256 + 333, 15 25.4 -> 26.9; 256 + 480, 20 32.5 -> 33.0; d = 64, 256 + 336, 15 15.0 -> 16.1; 240 + 678,
// 31 27.2 -> 29.2.
inline bool copying_wavefronts(int d, unsigned attend_blocks, unsigned copy_blocks, unsigned tiles) {
  return tiles > 1 && attend_blocks + copy_blocks <= 190 + 28 * tiles && update_finds_units(d, attend_blocks, copy_blocks, tiles);
}

// Two key streams per workgroup from 384 tokens on.  d = 128: always.  d = 64: workgroups of two streams have a unit to themselves,
// also those that copy rows of the update, which one-stream workgroups have room for: not where these would wait, and below 12
// tiles one stream next to copying wavefronts is the faster one.  `update_blocks` counts the plan's update also for a launch
// without it, whose outputs have to be the same bits (such launches lose 6 to 10 % by that where the update is what decides).  One
// launch, one stream (the better of its forms) -> two, workgroups of attention + update, tiles: 256 + 0, 39 30.4 -> 27.2 us; 256 +
// 284, 39 29.9 -> 27.4; 256 + 256, 20 17.4 -> 16.2; 240 + 324, 31 24.2 -> 22.3; 192 + 576, 23 19.2 -> 18.2; 180 + 810, 36 31.5 -> 24.5;
// 192 + 384, 12 12.2 -> 12.0; but 256 + 288, 14 14.0 -> 15.4; 256 + 768, 23 22.7 -> 24.9; 240 + 640, 16 16.9 -> 20.5; 240 + 248, 12 12.5
// -> 13.6; 256 + 128, 8 9.7 -> 10.6; 192 + 0, 7 8.2 -> 8.8; 160 + 0, 8 8.8 -> 8.9.
inline bool two_key_streams(int d, unsigned attend_blocks, unsigned update_blocks, unsigned tiles) {
  return d == 128 || (tiles >= 12 && update_finds_units(d, attend_blocks, update_blocks, tiles));
}

}  // namespace rules
}  // namespace heatkv
