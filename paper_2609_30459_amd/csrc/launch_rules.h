// The launch shapes that the library chooses where the caller leaves them open.
// They never change the records. Host code without dependencies, so that the
// rules can be read and tested by themselves.
#pragma once

namespace vio {

// Whether a tracking wave takes two keypoints (a half each) instead of one, for a
// launch of up to n_items. Two are bound by half the waves' longer chains, one by
// instruction issue and by the rounds its waves come in: from about six items per
// SIMD on two are faster, and at five and six levels, where one keypoint's kernel
// takes 140 and 159 registers and so three waves to a SIMD, from three on, where
// these start a second round.
// Four levels, streams of 2 x 752x480 with 960 items: four 42.7 us with one and 46.5
// with two, six 61.5 and 58.1, twelve 101.8 and 93.6; mono 320x240 of 200 items,
// sixteen 32.9 and 35.4, 32 53.2 and 52.0. Five: three such streams 42.5 and 50.5,
// four 60.0 and 50.3, a 4 x 1280x720 rig of 3,140 items 52.2 and 50.4, of 4,240 61.0
// and 60.2, one of 10,560 items 128.8 and 114.6. Six: three streams 47.6 and 60.0,
// four 65.8 and 61.8.
inline bool two_keypoints_a_wave(int n_items, int n_cus, int levels) {
  return n_items > (levels >= 5 ? 12 : 24) * n_cus;
}

}  // namespace vio
