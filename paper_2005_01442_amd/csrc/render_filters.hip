// render_filters.hip -- the whole-image forward kernel with local lighting and
// with the filters of the paper's comparison (gfx950).
//
// Three wavefronts per SIMD leave each lane 168 registers.  The lit kernels spill 24 to
// 27 of them, the pre-classified ones of 16-bit voxels 6 to 14, the other filters none
// or one.
#include "render_march.h"

namespace vr {

hipError_t launch_render_variant(const RenderArgs &a, int group, uint32_t lds, hipStream_t s) {
  if (a.shaded) return launch_render_grouped<true, 0>(a, group, lds, s);
  switch (a.filter) {
  case 1: return launch_render_grouped<false, 1>(a, group, lds, s);
  case 2: return launch_render_grouped<false, 2>(a, group, lds, s);
  default: return launch_render_grouped<false, 3>(a, group, lds, s);
  }
}

}  // namespace vr
