// The launch shapes that the library chooses where the caller leaves them open.
// They never change the records. Host code without dependencies, so that the
// rules can be read and tested by themselves.
#pragma once
#include <cstddef>

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

// Level-0 tile edge of the pyramid and detector for a handle whose cameras have so
// many 64-px tiles: 32 px for few of them (up to about half the compute units) up to
// four levels. Above, a 32-px tile's apron and its 256 threads cost more than the
// larger number of workgroups gives (it stages 8.6 bytes a pixel at five levels and
// 24 at six, a 64-px one 3.9 and 8.8). 64 and 32 px: mono 160x120 (6 tiles) 6.3 and
// 5.7 us at three levels, 7.3 and 7.5 at four, 9.5 and 11.8 at five, 15.7 and 23.0 at
// six; 320x240 (20) 7.3 and 7.2, 7.9 and 7.7, 11.1 and 12.4, 20.3 and 28.0; 641x479
// (88) 7.9 and 7.8, 8.3 and 8.5, 11.5 and 14.5, 20.9 and 36.5; two 752x480 (192) 8.1
// and 7.9, 10.1 and 10.4, 14.2 and 15.7, 24.0 and 45.9.
inline int default_pyr_tile(int tiles64, int levels) { return tiles64 <= 128 && levels <= 4 ? 32 : 64; }

// Whether a tile's detection and levels run in a workgroup each (`split` workgroups
// in all) instead of one after the other in one (`joined`). Two stage the tile
// twice, but halve the chain while all of them have a place at once: to a compute
// unit as many as the chains of their threads and their LDS allow, by measurement.
// In one and in two, 64-px tiles of four levels: 240 (joined 160) 11.0 and 8.5 us,
// 288 (192) 10.7 and 10.1, 480 (320) 12.7 and 11.9, 576 (384) 13.3 and 13.8; but 480
// (240) 11.4 and 12.6: where the joined ones have a compute unit each, up to 1.5 to one.
// Five levels: 240 14.5 and 11.9, 288 14.2 and 15.2, 480 (240) 14.3 and 18.8; six: 240
// 23.7 and 21.3, 288 24.0 and 27.0. 32-px tiles: four levels, 900 10.6 and 9.3, 1,080
// 10.4 and 10.6; five, 720 15.9 and 15.6, 900 15.9 and 16.1; six, 390 31.0 and 29.3,
// 600 33.4 and 36.6.
inline bool split_pyramid(int split, int joined, int tile, int levels, int n_cus) {
  if (tile == 32) return split <= n_cus * (levels <= 4 ? 4 : levels == 5 ? 3 : 2);
  if (levels > 4) return split <= n_cus;
  return split <= 2 * n_cus && (joined > n_cus || 2 * split <= 3 * n_cus);
}

// Whether a stream's host images (camera_bytes each) go up camera by camera, each
// beside the staging of the next one, instead of all at once. Among other streams'
// their staging hides the uploads anyway and each launch costs the host. A frame
// pushed, at once and camera by camera: 2 x 320x240 59.5 and 61.7 us, 4 x 400x300 82.2 and
// 84.4, 2 x 480x360 68.8 and 68.9, 2 x 640x480 76.9 and 75.8, 2 x 752x480 84.1 and 81.4,
// 4 x 640x480 110 and 106, 2 x 1280x720 123 and 113, 4 x 1920x1200 465 and 367. Four
// streams staged and stepped, and with three steps in flight: 2 x 640x480 157 and 164, 87
// and 88, 4 x 640x480 246 and 270, 146 and 156, 2 x 1280x720 278 and 276, 184 and 195, 4 x
// 1920x1200 1,160 and 1,105, 804 and 840.
inline bool split_upload(size_t camera_bytes, int cameras, bool among) {
  return among ? camera_bytes * cameras >= ((size_t)3 << 19) : camera_bytes >= ((size_t)1 << 18);
}

}  // namespace vio
