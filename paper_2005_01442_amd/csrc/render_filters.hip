// render_filters.hip -- the whole-image forward kernel with local lighting and
// with the filters of the paper's comparison (gfx950).
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
