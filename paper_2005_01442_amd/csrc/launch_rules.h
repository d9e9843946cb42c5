// launch_rules.h -- how launches are cut into pieces: plain arithmetic, for the
// host and the kernels alike (no HIP types).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace vr {

// What the rays of a launch look like from the volume.
struct RayField {
  double pitch = 0.0;     // voxels between neighbouring rays (the largest of the views)
  double rays = 0.0;      // pixels of all views
  double crossing = 0.0;  // rays that cross the volume, about
  bool inside = false;    // a view's eye lies in the volume
  double cover = 0.0;     // area of the volume's silhouettes over the images' (above 1: a closer view)
};

// Add a view.  The distance between rays is taken at the depth of the volume's
// centre; where the eye is so close, or inside, that the far side lies more than
// three times as deep, at a third of that.  (At the centre alone, views from
// inside the volume counted as arbitrarily dense, although most of their samples
// lie in front of the eye: 512x512x400 to 256^2 at 90 degrees, two lanes 0.57, four
// 0.34 ms.)
template <class Vol, class Cam>
inline void add_view(RayField &f, const Vol &v, const Cam &c) {
  const double n[3] = {(double)v.nx, (double)v.ny, (double)v.nz};
  bool inside = c.proj != 0;
  double z = 0.0, half = 0.0, f2 = 0.0;  // (a camera's forward vector need not have length 1)
  for (int k = 0; k < 3; ++k) {
    z += (0.5 * (n[k] - 1.0) - c.eye[k]) * c.fwd[k];
    half += 0.5 * n[k] * std::abs(c.fwd[k]);
    f2 += c.fwd[k] * c.fwd[k];
    inside = inside && c.eye[k] >= -0.5 && c.eye[k] <= n[k] - 0.5;
  }
  z /= f2;
  half /= f2;
  const double rays = (double)c.W * c.H;
  const double p = c.proj == 0 ? 2.0 * std::max(c.hw / c.W, c.hh / c.H)
                               : 2.0 * std::max(std::max(z, (z + half) / 3.0), 0.0) * c.th / c.H;
  const double area = (std::abs(c.fwd[0]) * n[1] * n[2] + std::abs(c.fwd[1]) * n[0] * n[2] + std::abs(c.fwd[2]) * n[0] * n[1]) /
                      std::sqrt(f2);
  const double silhouette = p > 0.0 ? area / (p * p) : 0.0;  // (p = 0: the volume lies behind the eye)
  const double before = f.rays;
  f.rays += rays;
  f.pitch = std::max(f.pitch, p);
  f.inside = f.inside || inside;
  f.crossing += std::min(rays, silhouette);
  f.cover = (f.cover * before + silhouette) / f.rays;
}

// Lanes per ray of a whole-image launch.  More lanes per ray make a wavefront's
// rays fewer and closer: its samples fit the LDS box at larger distances p between
// rays (8x4 rays of two samples up to p about 1.3, 4x4 of four up to 2.5, 2x2 of
// sixteen up to 5; a wavefront that does not fit gathers 16 rows per sample from
// global memory), and a launch of few rays is cut into more and shorter pieces;
// against that, each sample passes a longer compositing chain, and rays that miss
// the volume cost their lanes (about 0.035 ns a lane: 16 views of 512^2 that the
// volume covers to 5 %, p = 2.8: 1.07 ms with four, 2.56 with sixteen).  Measured in
// some 4000 launches (volumes of 64^3 to 1000x900x700, images of 40^2 to 1300^2, 1 to
// 16 views, framed, far, close, from inside, orthographic; the lines below are within
// 1 % of the best of 2, 4 and 16 lanes on average).  Step 0.5, int16, blocks and
// ERT, microseconds with 2 / 4 / 16 lanes:
//   256x256x200 to 128^2, framed, p = 3.7: 1220 / 510 / 151; 512^3 to 400^2, p = 2.5: 1880 / 730 / 600
//   256x256x200 to 256^2, framed, p = 1.9: 797 / 240 / 181; to 512^2, p = 0.9: 400 / 330 / 560
//   rays that all cross (a closer view): to 200^2, p = 0.8: 520 / 300 / 540, to 512^2, p = 0.3: 875 / 1085 / -
// When every ray crosses, two lanes fill the device evenly from about 61440 rays
// on; framed views, whose rays through the middle are the longest, gain from four
// up to some 150000 crossing rays, and where p is around 1, so that the box holds
// the samples of 8x4 rays only in part, beyond.  Longer steps need longer boxes and
// make shorter rays, which favours two lanes.  Time of two lanes over that of four,
// steps 0.5 / 0.75 / 1, volumes of 256^3 to 700x760x840:
//   p = 0.8, x = 145000: 1.06 / 0.99 / 0.93; p = 0.86, x = 420000: 0.94 / 0.89 / 0.84
//   p = 1.02, x = 260000: 1.01 / 0.96 / 0.91 (framed 1.08 / 1.03 / 0.96; fp32 1.02 / 0.96 / 0.91)
//   p = 1.05, x = 325000 or 640000: 1.05 / 0.98 / 0.91; p = 1.11 to 1.2, x = 260000 to 720000: 1.03 to 1.17 / 0.97 to 1.09 / 0.91 to 0.98
//   p = 1.34, x = 200000 or 560000: 1.2 / 1.2 / 1.2; without blocks the same and up to 0.2 more
// `full`: the rays of a closer view from which two lanes are ahead.  `heavy`: a
// sample costs several times a lookup of the box (pre-classification), which hides
// the chain: 256x256x200 to 512^2, close: 3.3 ms with two lanes, 2.9 with four;
// 700x760x840 to 700^2, close, p = 1.3: 1.07 times as long with two.
constexpr double kFullRays = 61440.0, kFullCells = 170000.0, kFullHeavy = 400000.0;
inline int ray_group(const RayField &f, double step, double full = kFullRays, bool heavy = false) {
  const double p = f.pitch, x = f.crossing, missing = f.rays - f.crossing;
  const double idle = heavy ? 4e6 : 1e6;  // missing rays that sixteen lanes are not worth
  if (missing > 12.0 * idle) return 2;
  if (p > 2.8) return missing > (p < 4.5 ? idle : 2.0 * idle) ? 4 : 16;
  const double few = 9300.0 * std::pow(std::max(1.0, p / 0.9), 1.45);
  if ((x <= few || ((p > 0.9 || heavy) && f.rays <= 20000.0)) && missing < (p <= 2.3 ? 0.15 * idle : idle)) return 16;
  if (p > 1.4) return 4;
  if (missing > 1.5e6) return 2;
  if (p > (heavy ? 1.08 : 1.2)) return 4;
  if (p > 1.08) return x > 200000.0 && step > 0.8 ? 2 : 4;
  if (f.cover < 2.0 && p >= 0.3) full = std::max(full, p > 0.95 && step <= 0.6 ? 300000.0 : (step <= 0.8 ? 150000.0 : 120000.0));
  return x > full ? 2 : 4;
}

// Lanes per ray of a pre-integrated launch: as above, and one where the rays fill
// the image closely and the device several times over (a cell's near value then
// is the lane's own of the step before).  One / two / four lanes, step 0.5,
// microseconds: 512x512x400 to 1024^2, p = 0.33: 5370 / 5820 / 6650, p = 0.93 (framed): - / 1640 / -;
// 128x120x100 to 700^2, p = 0.12: 897 / 955 / 1078; to 400^2, p = 0.2: 411 / 443 / 453;
// 256x256x200 to 400^2, p = 0.7: 800 / 560 / 514; to 256^2, close: 731 / 404 / 374.
inline int preint_group(const RayField &f, double step) {
  if (f.cover >= 1.0 && ((f.pitch < 0.6 && f.crossing > 300000.0) || (f.pitch < 0.22 && f.crossing > 147456.0))) return 1;
  return ray_group(f, step, kFullCells);
}

// Lanes per ray of a served request, which shares its launch with others: a
// launch of twelve requests fills the device whatever their size, and then has two
// workgroups per super-tile, eight parts each with sixteen lanes.  So sixteen
// are for small images and for coarse ones, and two from 200000 rays on (to
// 128^2, close, alone / twelve at once: 16 lanes 0.30 / 2.5 ms, 4 lanes 0.33 / 1.4 ms;
// to 400^2, close: 4 lanes 0.75 / 7.4 ms, 2 lanes 1.13 / 7.0 ms; to 512^2: 1.20 / 11.5, 0.99 / 9.2 ms).
inline int serve_group(const RayField &f) {
  const double p = f.pitch, x = f.crossing;
  if ((p > 2.8 && f.rays - x <= 2e6) || (p > 2.3 && x <= 20000.0 && f.rays - x < 150000.0) || (f.rays <= 20000.0 && x <= 10000.0)) return 16;
  return p > 1.08 || f.rays <= 200000.0 ? 4 : 2;
}

// Lanes per ray and scatter of the adjoint (render_bwd.hip): windows of LDS for
// 16 lanes each, over 4x4, 4x2 or 2x2 rays or one ray, placed for a whole step or
// for a ray's first samples, then its second ones; or one box per wavefront.
enum class Adjoint { k4x4, k4x2Step, k4x2Sample, k2x2Sample, k1, kBox };

// A window holds stencil bases up to 4 voxels apart in y and z, so the shape
// follows the rays' distance p and the step; launches of few rays take more lanes
// per ray, and long steps in dense launches the box, whose 32 rays share the
// cells that windows of 8 or 16 flush one by one.  Measured in some 700 launches (256x256x200,
// framed, near, far, inside, and 128^3 with 16 views; steps 0.5 to 8), relative to
// the box, for x crossing rays (4x4 / 4x2 by step / 4x2 by sample / 2x2 / one ray):
//   step 0.5, p = 0.6 to 0.85, x < 40000: 1.12 / 0.63 / 0.65 / 0.60 / 1.45; x > 100000: 0.78 / 0.62 / 0.65 / 0.72 / 2.2
//   step 0.5, p = 1.05, x > 300000: 0.71 / 0.52 / 0.55 / 0.67 / 2.2; p = 1.14: 1.56 / 0.74 / 0.68 / 0.58 / 1.8
//   step 0.5, p = 2.6: - / 0.92 / 1.0 / 0.05 / 0.08; p = 3.5, x < 10000: 1.6 / 0.86 / 1.0 / 0.18 / 0.07
//   step 1, p < 0.6, x < 100000: 1.0 / 0.92 / 0.94 / 1.6 / 5.3; x > 100000: 0.73 / 0.87 / 0.88 / 1.5 / 5.3
//   step 2, p < 0.6, x < 100000: 1.04 / 1.31 / 1.32 / 2.3 / 13 (the box: 0.94); x > 100000: 0.85 / 1.25 / 1.25 / 2.2 / 15
//   step 2, p = 0.9, x < 40000: 1.5 / 1.2 / 0.77 / 1.1 / 6; p = 1.05, x > 300000: 0.99 / 1.4 / 1.1 / 1.8 / 12 (the box: 0.90)
//   step 4, p < 0.6, x > 40000: 1.0 / 1.7 / 1.5 / 2.7 / 25 (the box: 0.92)
// (and rays that miss cost their lanes: 2048^2, one view a fortieth of it wide, 128x120x100, step 0.5:
// one ray 1.88 ms, 2x2 rays 1.19, the box 1.57; 4096^2 that miss, p = 1.14: 2x2 1.97, 4x2 1.57)
inline Adjoint adjoint_shape(const RayField &f, double step) {
  const double p = f.pitch, x = f.crossing, missing = f.rays - f.crossing;
  if (p > 2.9 && step <= 1.3 && missing <= 4e6) return Adjoint::k1;
  if (p > 1.25) return Adjoint::k2x2Sample;
  if (p > 1.08) {
    const bool dense = (x > 300000.0 && step > 0.9) || (x > 20000.0 && step > 1.2);
    return dense || missing > 8e6 ? Adjoint::k4x2Sample : Adjoint::k2x2Sample;
  }
  if (x <= 10000.0 || (x <= 20000.0 && step <= 1.2)) return Adjoint::k2x2Sample;
  if (step <= 0.8) return Adjoint::k4x2Step;
  if (x > 100000.0) {
    if (step <= 1.3) return p <= 0.6 ? Adjoint::k4x4 : Adjoint::k4x2Sample;
    return (p <= 0.9 && (step <= 3.0 || p > 0.4)) || step > 6.0 ? Adjoint::k4x4 : Adjoint::kBox;
  }
  if (p > 0.85 || x <= 20000.0) return Adjoint::k4x2Sample;
  if (x <= 40000.0 && step > 1.2) return step < 2.0 || (p > 0.6 && step < 3.0) ? Adjoint::k4x2Sample : Adjoint::kBox;
  if (x <= 40000.0) return Adjoint::k4x2Step;
  // (rays from an eye deep in the volume start side by side, on the same cells)
  return step <= 1.2 && !(f.inside && p < 0.6) ? Adjoint::k4x2Step : Adjoint::kBox;
}

// Lanes per ray where only the TF gradient is asked for: nothing is scattered, so
// the few rays and the coarse ones take more lanes, as in the forward, but each
// sample gathers its taps from global memory whatever their distance (2 / 4 / 16
// lanes, step 0.5, int16 256x256x200: to 256^2, framed, p = 1.9: 736 / 419 / 259 us, close,
// p = 0.7: 620 / 670 / 980; to 512^2, framed, p = 0.9: 753 / 625 / 739; 128^3 fp32, 16 views of
// 225^2, step 1: 867 / 1018 / 1594).  Long steps make short rays, which many lanes
// cut too small, and many close ones take one lane (step 4, to 1024^2, close:
// 1.12 ms with one, 1.45 with two; to 512^2, far, p = 2.8 with four 0.11, sixteen 0.15).
// Rays that miss cost their lanes (4096^2 of which 0.03 % cross, p = 2.3: 1.22 / 1.95 / 7.5 ms).
inline int tf_adjoint_group(const RayField &f, double step) {
  const double p = f.pitch, x = f.crossing, missing = f.rays - f.crossing;
  const double scale = step > 2.0 ? 0.36 : 1.0;
  if (missing > (p <= 1.0 ? 4e6 : 8e6)) return 2;
  if (x <= scale * (p > 1.9 ? 50000.0 : p > 0.7 ? 28000.0 : 10000.0) && missing < scale * 300000.0) return 16;
  if (p > 1.4) return 4;
  if (step > 1.5 && x > 150000.0 && p <= 0.6) return 1;
  if (x > 250000.0) return 2;
  return p > 1.0 || x <= 40000.0 || (f.cover < 2.0 && x <= 170000.0 && step <= 2.0) ? 4 : 2;
}

// `group`, or fewer lanes where a launch of `items` super-tile items (256 threads per
// lane of a ray's group, in whole rounds of eight) would have too many threads: HIP
// takes fewer than 2^32.  (32768 pixels along one edge, without a launch order, are
// padded to 2^22 items: 2^32 threads with four lanes.)
inline int lanes_within(int group, int64_t items) {
  while (group > 2 && ((items + 7) / 8 * 8) * 256 * group >= ((int64_t)1 << 32)) group = group > 4 ? 4 : 2;
  return group;
}

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
