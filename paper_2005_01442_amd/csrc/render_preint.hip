// render_preint.hip -- pre-integrated classification (gfx950).
//
// The paper pairs its ray caster with tables of previously integrated
// rendering (Section 2, the proposed method; the conclusion names
// pre-integrated rendering against sampling artefacts).  A ray segment of one
// step along which the value rises linearly from TF node i to node j has the
// emission-absorption integrals
//   alpha = 1 - exp(-tau(step)),  C = integral c(u(x)) sigma(u(x)) exp(-tau(x)) dx,
// tau(x) = integral_0^x sigma(u(x')) dx', u(x) = i + (j - i) x / step.
// k_preint_table tabulates them for every node pair; k_render_preint walks
// the lattice cells (between the boundaries t = k step and (k+1) step, the
// cells whose midpoints are the post-classified samples), reconstructs the
// value at each boundary once, and composites each cell with the table's
// bilinear lookup at (u(front), u(back)).
#include "vr_internal.h"

namespace vr {

// ---------------------------------------------------------------------------
// Table, FP64.  The segment of entry (i, j) is split where u crosses a node
// (sigma and c are linear between) into n = |j - i| pieces of length h = step / n.
// A piece's own integrals -- its emission G (attenuated from its front only) and
// its optical depth -- depend on its two nodes, h and the direction, not on the
// entry, so a workgroup takes all entries of one n and one direction: each piece
// is integrated once (sub-intervals of optical depth <= 1/32, 4-point
// Gauss-Legendre, tau exact, until its own depth passes 60), and an entry then
// composes its n pieces back to front, C = G + exp(-tau_piece) C.  That takes
// 2 K^2 piece integrations and K^3 / 3 compositions of three multiply-adds; one
// thread per entry integrated K^3 / 3 pieces, its longest thread 255 pieces of
// four exponentials one after another, on one wavefront per SIMD (K = 256: 205
// us, bound by that chain; 21 us now).
// ---------------------------------------------------------------------------
struct Piece {
  double g[3], t, depth;  // emission, exp(-depth), optical depth
};

// From node a to node b over length h.
__device__ inline Piece integrate_piece(const float4 &na, const float4 &nb, double h) {
  const double a[4] = {na.x, na.y, na.z, na.w}, b[4] = {nb.x, nb.y, nb.z, nb.w};
  // 4-point Gauss-Legendre on [-1, 1]
  const double gx[4] = {-0.8611363115940526, -0.3399810435848563, 0.3399810435848563, 0.8611363115940526};
  const double gw[4] = {0.3478548451374538, 0.6521451548625461, 0.6521451548625461, 0.3478548451374538};
  Piece p;
  p.g[0] = p.g[1] = p.g[2] = 0.0;
  p.depth = 0.5 * (a[3] + b[3]) * h;
  p.t = exp(-p.depth);
  const double ds = (b[3] - a[3]) / h;  // d sigma / dx
  const int sub = max(1, (int)ceil(p.depth * 32.0));
  const double w0 = h / (double)sub;
  for (int q = 0; q < sub; ++q) {
    const double x0 = q * w0;
    if (a[3] * x0 + 0.5 * ds * x0 * x0 > 60.0) break;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const double x = x0 + 0.5 * w0 * (1.0 + gx[g]);
      const double w = x / h;
      const double sg = a[3] + ds * x;
      const double f = 0.5 * w0 * gw[g] * sg * exp(-(a[3] * x + 0.5 * ds * x * x));
#pragma unroll
      for (int c = 0; c < 3; ++c) p.g[c] += ((1.0 - w) * a[c] + w * b[c]) * f;
    }
  }
  return p;
}

// Workgroup 0: the diagonal; 2 n - 1 and 2 n: the entries (i, i + n) and
// (i + n, i).  LDS: five arrays of K - 1 doubles.
__global__ __launch_bounds__(256) void k_preint_table(const float *tf, int K, double step, float4 *out,
                                                     uint32_t *status) {
  extern __shared__ __attribute__((aligned(16))) double pieces[];
  const float4 *node = reinterpret_cast<const float4 *>(tf);
  // an invalid node anywhere makes the whole table NaN (and is recorded)
  int bad = 0;
  for (int j = threadIdx.x; j < K; j += 256) bad |= tf_node_valid(node[j]) ? 0 : 1;
  bad = __syncthreads_or(bad);
  if (bad && threadIdx.x == 0 && status) __hip_atomic_store(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int n = ((int)blockIdx.x + 1) / 2;
  const bool down = blockIdx.x != 0 && blockIdx.x % 2 == 0;
  if (n == 0 || bad) {
    for (int i = threadIdx.x; i < K - n; i += 256) {
      float4 e = nan_rgba();
      if (!bad) {
        const float4 c = node[i];
        const double a = -expm1(-(double)c.w * step);
        e = make_float4((float)(c.x * a), (float)(c.y * a), (float)(c.z * a), (float)a);
      }
      out[down ? (size_t)(i + n) * K + i : (size_t)i * K + i + n] = e;
    }
    return;
  }
  const int np = K - 1;
  double *g0 = pieces, *g1 = g0 + np, *g2 = g1 + np, *tr = g2 + np, *dp = tr + np;
  const double h = step / (double)n;
  for (int q = threadIdx.x; q < np; q += 256) {
    const Piece p = integrate_piece(node[down ? q + 1 : q], node[down ? q : q + 1], h);
    g0[q] = p.g[0];
    g1[q] = p.g[1];
    g2[q] = p.g[2];
    tr[q] = p.t;
    dp[q] = p.depth;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < K - n; i += 256) {
    // back to front: up, pieces i + n - 1 .. i; down, pieces i .. i + n - 1
    double c0 = 0.0, c1 = 0.0, c2 = 0.0, tau = 0.0;
    int q = down ? i : i + n - 1;
    const int dq = down ? 1 : -1;
#pragma unroll 4
    for (int m = 0; m < n; ++m, q += dq) {
      const double t = tr[q];
      c0 = fma(t, c0, g0[q]);
      c1 = fma(t, c1, g1[q]);
      c2 = fma(t, c2, g2[q]);
      tau += dp[q];
    }
    out[down ? (size_t)(i + n) * K + i : (size_t)i * K + i + n] =
        make_float4((float)c0, (float)c1, (float)c2, (float)(-expm1(-tau)));
  }
}

hipError_t launch_preint_table(const float *tf, int K, float step, float4 *out, uint32_t *status, hipStream_t s) {
  const uint32_t lds = 5u * (uint32_t)(K - 1) * 8u;  // at most 41 KB
  hipLaunchKernelGGL(k_preint_table, dim3((unsigned)(2 * K - 1)), dim3(256), lds, s, tf, K, (double)step, out, status);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Render.
// ---------------------------------------------------------------------------

// Bilinear lookup of the table at node coordinates (uf, ub), clamped.
__device__ inline float4 preint_lookup(const float4 *tab, int K, float uf, float ub) {
  uf = fminf(fmaxf(uf, 0.0f), (float)(K - 1));
  ub = fminf(fmaxf(ub, 0.0f), (float)(K - 1));
  const int i = min((int)uf, K - 2), j = min((int)ub, K - 2);
  const float wf = uf - (float)i, wb = ub - (float)j;
  const float4 *r0 = tab + (size_t)i * K + j;
  const float4 p00 = r0[0], p01 = r0[1], p10 = r0[K], p11 = r0[K + 1];
  float4 o;
  o.x = fmaf(wf, fmaf(wb, p11.x - p10.x, p10.x) - fmaf(wb, p01.x - p00.x, p00.x), fmaf(wb, p01.x - p00.x, p00.x));
  o.y = fmaf(wf, fmaf(wb, p11.y - p10.y, p10.y) - fmaf(wb, p01.y - p00.y, p00.y), fmaf(wb, p01.y - p00.y, p00.y));
  o.z = fmaf(wf, fmaf(wb, p11.z - p10.z, p10.z) - fmaf(wb, p01.z - p00.z, p00.z), fmaf(wb, p01.z - p00.z, p00.z));
  o.w = fmaf(wf, fmaf(wb, p11.w - p10.w, p10.w) - fmaf(wb, p01.w - p00.w, p00.w), fmaf(wb, p01.w - p00.w, p00.w));
  return o;
}

// Lane j - 1's value to lane j of a ray group (lane 0 keeps `first`).
template <int G>
__device__ inline int from_left(int x, int first) {
  if constexpr (G == 1) return first;
  // quad_perm [0, 0, 2, 2] / [0, 0, 1, 2], row_shr:1
  constexpr int ctrl = G == 2 ? 0xA0 : (G == 4 ? 0x90 : 0x111);
  const int y = __builtin_amdgcn_mov_dpp(x, ctrl, 0xF, 0xF, true);
  return threadIdx.x % G == 0 ? first : y;
}
// Lane j + 1's value to lane j of a ray group (the last lane gets 0).
template <int G>
__device__ inline int from_right(int x) {
  if constexpr (G == 1) return 0;
  // quad_perm [1, 1, 3, 3] / [1, 2, 3, 3], row_shl:1
  constexpr int ctrl = G == 2 ? 0xF5 : (G == 4 ? 0xF9 : 0x101);
  const int y = __builtin_amdgcn_mov_dpp(x, ctrl, 0xF, 0xF, true);
  return threadIdx.x % G == G - 1 ? 0 : y;
}

// Walk the boundary points k = k0 .. k0 + ns of a ray with the wavefront in
// step, a group of G lanes per ray (as walk_group does for samples): lane j
// takes point k + j, and the cell it closes, k + j - 1, has its front at lane
// j - 1's point (lane 0's at the last point of the step before).  Skipping: a cell
// is skipped iff no value in the union of its two points' block ranges meets
// extinction (its ramp then integrates to exactly zero).  A point is
// reconstructed once, when a cell of its step needs it; a cell whose front the
// step before did not reconstruct has it reconstructed first.  The group's cells
// are then composited front to back by every lane in the one-lane march's
// operations and order (a cell not taken enters as the identity), so the image
// does not depend on G.  When no lane closes a cell the wavefront leaps (points up
// to the leap target stay in the current, empty, block, so every skipped cell
// lies in one empty block).
template <int G, int DT>
__device__ inline float4 march_preint(const VolConst &v, const TfShared &s, const TfConst &tf, const MarchConst &mc,
                                      const float4 *tab, const Ray &r0, __amdgpu_buffer_rsrc_t rs, ValBox &box,
                                      uint32_t &evaluated, uint32_t &unstaged) {
  Ray r = r0;
  r.s0 = r0.s0 - 0.5f * mc.step;  // boundary point k sits at s0 + (k - k0) step - step/2
  const int j = (int)(threadIdx.x % G);
  const bool ert_on = mc.ert > 0.0f && mc.ert < 1.0f;
  const int kb = r.hit ? r.k0 : 0x7fffffff;
  const int ke = r.hit ? r.k0 + r.ns + 1 : 0;
  bool alive = r.hit;
  int k = wave_min_i32(kb);
  const int kend = wave_max_i32(ke);
  int kfree = kb;  // points below kfree: before the ray, or left in an empty block
  // the grid constants of the block lookup and leap pinned in scalar
  // registers, so the loop does not re-read them from the kernel arguments
  // (vector registers would exceed this kernel's budget)
  VolConst vg = v;
  {
    int a0 = __builtin_amdgcn_readfirstlane(vg.nx), a1 = __builtin_amdgcn_readfirstlane(vg.ny),
        a2 = __builtin_amdgcn_readfirstlane(vg.nz), a3 = __builtin_amdgcn_readfirstlane(vg.edge_shift),
        a4 = __builtin_amdgcn_readfirstlane(vg.nbx), a5 = __builtin_amdgcn_readfirstlane(vg.nby);
    asm volatile("" : "+s"(a0), "+s"(a1), "+s"(a2), "+s"(a3), "+s"(a4), "+s"(a5));
    vg.nx = a0;
    vg.ny = a1;
    vg.nz = a2;
    vg.edge_shift = a3;
    vg.nbx = a4;
    vg.nby = a5;
  }
  int cb = -1;        // block of this lane's last point, and whether it is occupied
  bool cocc = false;
  int last_block = 0;        // block << 1 | occupied of the group's point k - 1, when it is `carried`
  bool carried = false;      // (uniform over the wavefront)
  int klast = -0x7fffffff;   // the group's last reconstructed point and its value
  float vlast = 0.0f;
  float C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, T = 1.0f;
  auto value_at = [&](float px, float py, float pz) -> float {
    Stencil st = make_stencil(px, py, pz);
    if (box.valid) return reconstruct_box(box, st);
    ++unstaged;
    return reconstruct<DT>(rs, v, st);
  };
  while (k < kend) {
    const int kk = k + j;
    const bool in = alive && kk >= kfree && kk < ke;
    bool want = in && kk > kb;
    float px, py, pz;
    lattice_point(r, mc.step, kk, px, py, pz);
    int bc[3] = {0, 0, 0};
    if (mc.skip) {
      if (!carried) {  // after a leap: the block of the front of lane 0's cell
        float fx, fy, fz;
        lattice_point(r, mc.step, k - 1, fx, fy, fz);
        const int b = block_of(vg, fx, fy, fz, bc);
        last_block = b << 1 | (block_occupied(v, s, tf, b) ? 1 : 0);
      }
      const int b = block_of(vg, px, py, pz, bc);
      if (b != cb) {
        cb = b;
        cocc = block_occupied(v, s, tf, b);
      }
      const int here = cb << 1 | (cocc ? 1 : 0);
      const int front = from_left<G>(here, last_block);
      last_block = G == 1 ? here : from_group_lane_i32<G, G - 1>(here);
      carried = true;
      if (want && !cocc && !(front & 1))  // two empty blocks: empty only if the union of their ranges is
        want = front != here &&
               range_occupied(s, tf.K, tf.v0, tf.scale, fminf(v.minmax[front >> 1].x, v.minmax[cb].x),
                              fmaxf(v.minmax[front >> 1].y, v.minmax[cb].y));
    }
    if (__ballot(want) == 0ull) {
      int prop = 0x7fffffff;
      if (in) {
        if (mc.skip && !cocc) {
          kfree = leap_target(vg, r, bc, mc.step, kk);
          prop = kfree;
        } else {
          prop = kk + 1;
        }
      } else if (alive && kk < ke) {
        prop = kfree;
      }
      const int m = wave_min_i32(prop);
      carried = m <= k + G;
      k = m > k + G ? m : k + G;
      continue;
    }
    // the point is the back of this lane's cell or the front of the next lane's
    const int next_wants = from_right<G>(want ? 1 : 0);  // (every lane takes part in the exchange)
    const bool need = want || next_wants != 0;
    const bool need_front = want && j == 0 && klast != k - 1;
    float vfront = vlast;
    if (__ballot(need_front) != 0ull) {
      float fx = 0.0f, fy = 0.0f, fz = 0.0f;
      if (need_front) lattice_point(r, mc.step, k - 1, fx, fy, fz);
      if (box.cells) vbox_prepare<DT>(box, rs, v, r, need_front, fx, fy, fz);
      if (need_front) vfront = value_at(fx, fy, fz);
    }
    if (box.cells) vbox_prepare<DT>(box, rs, v, r, need, px, py, pz);
    float vcur = 0.0f;
    if (need) vcur = value_at(px, py, pz);
    vfront = __builtin_bit_cast(float, from_left<G>(__builtin_bit_cast(int, vcur), __builtin_bit_cast(int, vfront)));
    float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);  // the identity unless taken
    if (want) q = preint_lookup(tab, tf.K, (vfront - tf.v0) * tf.scale, (vcur - tf.v0) * tf.scale);
    bool live = alive;
    auto link = [&](auto I_) {
      constexpr int I = decltype(I_)::value;
      const float x = from_group_lane<G, I>(q.x), y = from_group_lane<G, I>(q.y), z = from_group_lane<G, I>(q.z);
      const float w = from_group_lane<G, I>(q.w);
      if (j == I && want && live) ++evaluated;
      const float Tl = live ? T : 0.0f;
      C0 = fmaf(Tl, x, C0);
      C1 = fmaf(Tl, y, C1);
      C2 = fmaf(Tl, z, C2);
      T = T * (1.0f - (live ? w : 0.0f));
      if (ert_on && (1.0f - T) >= mc.ert) live = false;
    };
    for_each_index<G>(link);
    alive = live;
    vlast = from_group_lane<G, G - 1>(vcur);
    klast = from_group_lane_i32<G, G - 1>(need ? k + G - 1 : -0x7fffffff);
    k += G;
  }
  return make_float4(C0, C1, C2, 1.0f - T);
}

// One wavefront item of the pre-integrated render: wavefront w of workgroup item
// i (a part of a super-tile).
template <int G, int DT>
__device__ inline void preint_wave_item(const RenderArgs &a, const TfShared &s, bool tf_ok, const float4 *tab,
                                        ValBox &box, __amdgpu_buffer_rsrc_t rs, int64_t i, int w, uint32_t &evaluated,
                                        uint32_t &unstaged, uint32_t &lattice, uint32_t &hits) {
  int part;
  const SuperTile st = group_tile_of<G>(a.order, i, a.W, a.H, a.n_views, a.chunk_edge, part);
  if (!st.valid) return;  // uniform over the wavefront
  int col, row;
  group_pixel_of<G>(st.sx, st.sy, part, w * kWaveSize + (int)(threadIdx.x % kWaveSize), col, row);
  const bool inside = col < a.W && row < a.H;
  const bool lead = threadIdx.x % G == 0;  // the lane that stores its group's pixel
  if (!tf_ok) {
    if (inside && lead) reinterpret_cast<float4 *>(a.out)[((size_t)st.view * a.H + row) * a.W + col] = nan_rgba();
    return;
  }
  const CamConst &cam = a.cams[st.view];
  Ray r;
  r.hit = false;
  r.ns = 0;
  r.k0 = 0;
  r.s0 = 0.0f;
  if (inside) r = setup_ray(cam, col, row, a.vol.nx, a.vol.ny, a.vol.nz, a.mc.step);
  const float4 rgba = march_preint<G, DT>(a.vol, s, a.tf, a.mc, tab, r, rs, box, evaluated, unstaged);
  if (inside && lead) reinterpret_cast<float4 *>(a.out)[((size_t)st.view * a.H + row) * a.W + col] = rgba;
  lattice += lead ? (uint32_t)r.ns : 0u;
  hits += lead && r.hit ? 1u : 0u;
}

// Queued like the whole-image forward (one workgroup item per workgroup without
// queue counters); registers budgeted for three wavefronts per SIMD, which
// the LDS value boxes allow.
template <int G, int DT>
__global__ __launch_bounds__(kWgSize) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_render_preint(
    const RenderArgs args, const float4 *tab) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const RenderArgs &a = kernarg<RenderArgs>();
  if (!a.queue) {
    int part;
    if (!group_tile_of<G>(a.order, blockIdx.x, a.W, a.H, a.n_views, a.chunk_edge, part).valid)
      return;  // uniform over the workgroup
  }
  TfShared s = carve_tf(lds, a.tf.K);
  if (a.occ_lds_words > 0)
    stage_occupancy(s, a.vol, lds + vbox_lds_offset(a.tf.K) + vbox_lds_bytes(), a.occ_lds_words);
  const bool tf_ok = load_tf(s, a.tf);
  __amdgpu_buffer_rsrc_t rs = make_rsrc(a.vol.data, a.vol.bytes);
  ValBox box;
  box.valid = false;
  box.ox = box.oy = box.oz = 0;
  box.cells = a.use_box ? reinterpret_cast<float *>(lds + vbox_lds_offset(a.tf.K)) + (threadIdx.x / kWaveSize) * kVBoxCells
                        : nullptr;
  uint32_t evaluated = 0, unstaged = 0, lattice = 0, hits = 0;
  if (!a.queue) {
    preint_wave_item<G, DT>(a, s, tf_ok, tab, box, rs, blockIdx.x, (int)(threadIdx.x / kWaveSize), evaluated,
                         unstaged, lattice, hits);
  } else {
    const int x = (int)(blockIdx.x % kXcds);
    int w = 0;
    int64_t i = 0;
    while (next_wave_item(a.queue, (uint32_t)a.queue_items, x, i, w))
      preint_wave_item<G, DT>(a, s, tf_ok, tab, box, rs, i, w, evaluated, unstaged, lattice, hits);
  }
  if (a.counters) {
    wave_count(a.counters + 0, evaluated);
    wave_count(a.counters + 1, lattice);
    wave_count(a.counters + 2, hits);
    wave_count(a.counters + 3, unstaged);
  }
}

template <int G>
static hipError_t launch_preint_as(const RenderArgs &a0, const float4 *tab, uint32_t lds, hipStream_t s) {
  RenderArgs a = a0;
  int64_t grid = group_grid(render_grid(a), G);
  auto *k = a.vol.dtype == kU16 ? &k_render_preint<G, kU16> : (a.vol.dtype == kI16 ? &k_render_preint<G, kI16> : &k_render_preint<G, kF32>);
  const void *fn = reinterpret_cast<const void *>(k);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  a.queue = nullptr;
  a.queue_items = 0;
  if (a.order) {
    const int64_t resident = resident_workgroups(fn, lds);
    if (resident >= kXcds && resident < grid) {
      a.queue = reinterpret_cast<uint32_t *>(const_cast<int32_t *>(a.order) + tile_order_count(a));
      a.queue_items = (int32_t)(grid / kXcds * kWavesPerWg);
      grid = resident;
    }
  }
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kWgSize), lds, s, a, tab);
  return hipGetLastError();
}

hipError_t launch_render_preint(const RenderArgs &a0, const float4 *tab, hipStream_t s) {
  RenderArgs a = a0;
  uint32_t lds = tf_lds_bytes(a.tf.K);
  const uint32_t with_box = vbox_lds_offset(a.tf.K) + vbox_lds_bytes();
  a.use_box = with_box <= max_lds_per_workgroup() ? 1 : 0;
  if (a.use_box) lds = with_box;
  a.occ_lds_words = a.use_box ? occupancy_lds_words(a.vol, lds) : 0;
  lds += (uint32_t)a.occ_lds_words * 4u;
  switch (lanes_within(preint_group(ray_field(a), a.mc.step), render_grid(a))) {
  case 16: return launch_preint_as<16>(a, tab, lds, s);
  case 4: return launch_preint_as<4>(a, tab, lds, s);
  case 1: return launch_preint_as<1>(a, tab, lds, s);
  default: return launch_preint_as<2>(a, tab, lds, s);
  }
}

}  // namespace vr
