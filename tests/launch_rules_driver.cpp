// The launch rules of csrc/launch_rules.h as C functions, for test_launch_rules.py.
#include "launch_rules.h"

namespace {
struct Vol {
  int32_t nx, ny, nz;
};
struct Cam {
  double eye[3], fwd[3], th, hw, hh;
  int32_t proj, W, H;
};

// `views` equal views; cam: eye, forward, tan(fov / 2) (perspective) or half extents (orthographic).
vr::RayField field(const int32_t *dims, const double *cam, int proj, int W, int H, int views) {
  const Vol v{dims[0], dims[1], dims[2]};
  const Cam c{{cam[0], cam[1], cam[2]}, {cam[3], cam[4], cam[5]}, cam[6], cam[7], cam[8], proj, W, H};
  vr::RayField f;
  for (int i = 0; i < views; ++i) vr::add_view(f, v, c);
  return f;
}
}  // namespace

extern "C" {
int64_t serve_blocks(int64_t items, int parts) { return vr::serve_blocks(items, parts); }
void serve_part(int64_t block, int parts, int64_t *item, int *part) {
  const vr::ServePart p = vr::serve_part_of(block, parts);
  *item = p.item;
  *part = p.part;
}
void ray_field(const int32_t *dims, const double *cam, int proj, int W, int H, int views, double *out) {
  const vr::RayField f = field(dims, cam, proj, W, H, views);
  out[0] = f.pitch;
  out[1] = f.rays;
  out[2] = f.crossing;
  out[3] = f.cover;
}
int ray_group(const int32_t *dims, const double *cam, int proj, int W, int H, int views, double step, int heavy) {
  return vr::ray_group(field(dims, cam, proj, W, H, views), step, heavy ? vr::kFullHeavy : vr::kFullRays, heavy != 0);
}
int lanes_within(int group, int64_t items) { return vr::lanes_within(group, items); }
int preint_group(const int32_t *dims, const double *cam, int proj, int W, int H, int views, double step) {
  return vr::preint_group(field(dims, cam, proj, W, H, views), step);
}
int adjoint_shape(const int32_t *dims, const double *cam, int proj, int W, int H, int views, double step) {
  return (int)vr::adjoint_shape(field(dims, cam, proj, W, H, views), step);
}
int tf_adjoint_group(const int32_t *dims, const double *cam, int proj, int W, int H, int views, double step) {
  return vr::tf_adjoint_group(field(dims, cam, proj, W, H, views), step);
}
int serve_group(const int32_t *dims, const double *cam, int proj, int W, int H) {
  return vr::serve_group(field(dims, cam, proj, W, H, 1));
}
}
