// launch_rules.h -- how launches are cut into pieces: plain arithmetic, for the
// host and the kernels alike (no HIP types).
#pragma once

#include <stdint.h>

namespace vr {

// Workgroup -> (item, part) of a serving launch with `parts` workgroups per
// item: the parts of item i run on XCD i mod 8 (the hardware hands workgroup b
// to XCD b mod 8), eight items side by side and their parts one after another.
// A request marched by fewer lanes per ray than `parts` leaves its last parts
// empty, on every XCD alike.  (Parts side by side put the working ones of a
// launch of 256 items, four of eight, on half of the XCDs: a 256x256 request
// close to a 256x256x200 volume took 0.73 ms, 0.46 now.)
constexpr int kServeXcds = 8;
struct ServePart {
  int64_t item;
  int part;
};
constexpr ServePart serve_part_of(int64_t block, int parts) {
  const int64_t run = kServeXcds * (int64_t)parts;
  return {block / run * kServeXcds + block % kServeXcds, (int)(block / kServeXcds % parts)};
}
// Workgroups of such a launch: the last eight items are padded.
constexpr int64_t serve_blocks(int64_t items, int parts) { return (items + kServeXcds - 1) / kServeXcds * kServeXcds * parts; }

}  // namespace vr
