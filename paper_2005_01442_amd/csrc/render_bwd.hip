// render_bwd.hip -- adjoint of the forward ray caster (gfx950).
//
// Forward model per ray: C = sum_k T_k a_k c_k, T_{k+1} = T_k (1 - a_k),
// A = 1 - T_end, a_k = 1 - exp(-sigma_k step).  For L with g = dL/d(C, A):
//   dL/dc_k     = g_C T_k a_k
//   dL/dsigma_k = step (g_C . (T_{k+1} c_k - S_k) + g_A T_end),
//   S_k = sum_{m>k} T_m a_m c_m = C_end - C_{<=k},
// then through the TF segment (node difference x (K-1)/(v1-v0), zero where u
// was clamped) to the value, and through the 64 B-spline weights to the
// voxels.  The march is recomputed front to back with the forward's exact
// arithmetic, so C_{<=k}, T_k and the early-termination sample are the
// forward's; C_end and T_end come from the saved forward image.  Nothing per
// sample is stored.
#include <algorithm>

#include "vr_internal.h"

namespace vr {

// dv * w_a w_b w_c onto the 64 taps (clamped taps pile onto edge voxels).
__device__ inline void scatter_taps(float *g, const VolConst &v, const Stencil &st, float dv) {
  int xs[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) xs[a] = min(max(st.ix - 1 + a, 0), v.nx - 1);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t z = (uint32_t)min(max(st.iz - 1 + c, 0), v.nz - 1);
    float wc = dv * st.wz[c];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      uint32_t y = (uint32_t)min(max(st.iy - 1 + b, 0), v.ny - 1);
      uint32_t rowb = (z * (uint32_t)v.ny + y) * (uint32_t)v.nx;
      float wb = wc * st.wy[b];
#pragma unroll
      for (int a = 0; a < 4; ++a) unsafeAtomicAdd(g + rowb + (uint32_t)xs[a], wb * st.wx[a]);
    }
  }
}

// ---------------------------------------------------------------------------
// Gradient windows.  A wavefront's samples of one step fall into four groups of
// 16 lanes (a DPP row: 16 / G neighbouring rays, G samples each), and each
// group accumulates its grid gradient in a 12 x 8 x 8 window of LDS (x, y, z),
// addressed toroidally (a voxel's slot is its coordinate modulo the extent):
// when the group's stencils leave the window, it moves, and only the cells that
// drop out are added to global memory (one atomic per touched voxel) and
// cleared.  The window moves by single planes in y and z, and in x by aligned
// quads of voxels: atomics on single x-planes, every lane in a cache line of its
// own, took 100 ms of a 297 ms step (256^3 fp32, 64 views of 512^2).
//
// The 64 taps of a sample are dv wx_a wy_b wz_c.  In round r of a step the
// sample of lane r of every group is applied by the group's 16 lanes: lane
// (a = l mod 4, c = l / 4) holds x tap a and z tap c and walks the four y taps,
//   cell(a, b, c) += (dv wx_a wz_c) wy_b.
// The lane's product comes through LDS (staged by the sample's lane: a
// transpose per group, half of its samples at a time), wy_b and the sample's
// place in the window arrive as DPP row broadcasts inside the multiply-adds and
// address adds.  The taps of one sample are distinct cells and the groups'
// windows are distinct memory, so plain read-add-write is exact; rounds follow
// each other in LDS order.
//
// What bounds it: LDS and VALU issue per sample.  Four samples share a round of
// 14 VALU and 9 LDS instructions (64 lanes each); one sample per wavefront
// round, 64 lanes on its 64 taps, took 13.5 VALU and 5 LDS instructions per
// sample and one LDS round trip per two (256^3 fp32, 64 views of 512^2, forward
// and adjoint: 251 ms, then 167 ms; 512x512x400 int16 to 1024^2: 9.1, then 6.9
// ms).  LDS float atomics (ds_add_f32) would take one lane per ~3 cycles, also
// without conflicts.
//
// Slots lie at x + 12 z + 96 y (dwords): the 16 lanes of a group hit 16
// distinct banks.  Coordinates are those of the unclamped stencil; flushing
// clamps them to the grid, so edge stencils need no path of their own.
// ---------------------------------------------------------------------------
constexpr int kWinX = 12, kWin = 8;                 // window extent in x, and in y and z
constexpr int kWinZ = kWinX, kWinY = kWinX * kWin;  // strides of z and y
constexpr int kWinCells = kWinX * kWin * kWin; // of one group
constexpr int kRows = kWaveSize / 16;          // groups of a wavefront
constexpr int kSpread = kWin - 4;              // stencil bases of a group may differ by this much in y and z,
constexpr int kSpreadX = kWinX - 4;            // and lie this far from the window's x origin
// staged products (of at most 8 samples per group at once): 16 per sample, 20 dwords apart and the groups 176 (48 modulo
// 64 banks), so that the 16-byte writes and the groups' reads spread over banks
constexpr int kProdLane = 20, kProdRow = 8 * kProdLane + 16;
constexpr int kWinFloats = kRows * kWinCells, kProdFloats = kRows * kProdRow;

typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
__device__ inline lds_float *lds_at(uint32_t address) { return (lds_float *)(uintptr_t)address; }
__device__ inline uint32_t lds_address(lds_float *p) { return (uint32_t)(uintptr_t)p; }

// LDS layout of the adjoint: TF + prefix counts, TF gradient (four planes of K
// doubles, when requested), then 16-byte aligned per-wavefront windows, or the
// box, and staging areas; with up to 256 nodes two workgroups fit a CU.
//
// The TF gradient is in doubles because ds_add_f64 is the faster atomic: with 64
// lanes on distinct words it takes the LDS 9 cycles, ds_add_f32 179 (one lane
// after the other).  In floats, two copies by lane parity, the adds took 27 of
// 167 ms (256^3 fp32, 64 views of 512^2, forward and adjoint; 140 ms now) and
// 0.3 of 6.9 ms (512x512x400 int16 to 1024^2).  Planes per component put
// neighbouring nodes on neighbouring banks.
__host__ __device__ inline uint32_t tf_grad_bytes(int K, bool with_tf_grad) {
  return with_tf_grad ? (uint32_t)K * 4u * (uint32_t)sizeof(double) : 0u;
}
__host__ __device__ inline uint32_t grid_lds_offset(int K, bool with_tf_grad) {
  return (tf_lds_bytes(K) + tf_grad_bytes(K, with_tf_grad) + 15u) & ~15u;
}
typedef __attribute__((address_space(3))) double lds_double;

struct GradWindow {
  lds_float *cells;  // this lane's group's window, zero outside use; nullptr: no windows
  lds_float *prod;   // this lane's group's staged products
  int lo[3];         // origin of the window, lo[0] a multiple of 4
  int sx;            // x slot of lo[0]: 0, 4 or 8
  int ahead;         // bit a: the group's rays run towards higher coordinates of axis a
  bool valid;        // (lo, sx, ahead and valid are uniform over the group)
};

__device__ inline int row_min_i32(int x) {
  x = min(x, __builtin_amdgcn_mov_dpp(x, kDppQuadSwap1, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_mov_dpp(x, kDppQuadSwap2, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_mov_dpp(x, kDppHalfMirror, 0xF, 0xF, false));
  return min(x, __builtin_amdgcn_mov_dpp(x, kDppMirror, 0xF, 0xF, false));
}

__device__ inline uint32_t clamp_index(int x, int n) { return (uint32_t)min(max(x, 0), n - 1); }

// Add kWin cells, `stride` apart, to global memory and clear them: the cells of
// slots t = 0 .. 7 along an axis of n voxels whose window starts at lo, its
// voxels `pitch` apart in the grid.  All cells are read before the first is
// used (one LDS round trip); a cell's voxel is worked out only where it holds
// something (worked out incrementally for every cell: 512x512x400 int16 step
// 6.6 -> 7.0 ms, most of its cells being empty).
__device__ inline void win_flush_run(lds_float *c, int stride, float *grad, uint32_t base, int lo, int n, uint32_t pitch) {
  float val[kWin];
#pragma unroll
  for (int t = 0; t < kWin; ++t) val[t] = c[t * stride];
#pragma unroll
  for (int t = 0; t < kWin; ++t)
    if (val[t] != 0.0f) {
      unsafeAtomicAdd(grad + (base + clamp_index(lo + ((t - lo) & 7), n) * pitch), val[t]);
      c[t * stride] = 0.0f;
    }
}

// Flush plane p of the window in y (A = 1) or z (A = 2): twelve lanes along x.
template <int A>
__device__ inline void win_flush_plane(const GradWindow &w, float *grad, const VolConst &v, int p) {
  const int l = (int)(threadIdx.x % 16);
  if (l >= kWinX) return;
  const int xs = w.sx + l;  // slot of voxel lo[0] + l
  const uint32_t nx = (uint32_t)v.nx, nxy = nx * (uint32_t)v.ny, gx = clamp_index(w.lo[0] + l, v.nx);
  lds_float *c = w.cells + (xs >= kWinX ? xs - kWinX : xs);
  if constexpr (A == 1)
    win_flush_run(c + (p & 7) * kWinY, kWinZ, grad, gx + clamp_index(p, v.ny) * nx, w.lo[2], v.nz, nxy);
  else
    win_flush_run(c + (p & 7) * kWinZ, kWinY, grad, gx + clamp_index(p, v.nz) * nxy, w.lo[1], v.ny, nx);
}

// Flush the aligned quad of x planes p .. p + 3: four lanes along x, four z.
__device__ inline void win_flush_quad(const GradWindow &w, float *grad, const VolConst &v, int p) {
  const int l = (int)(threadIdx.x % 16);
  const uint32_t nx = (uint32_t)v.nx, nxy = nx * (uint32_t)v.ny, gx = clamp_index(p + (l & 3), v.nx);
  const int xs = w.sx + (p - w.lo[0]) + (l & 3);
  lds_float *c = w.cells + (xs >= kWinX ? xs - kWinX : xs);
#pragma unroll
  for (int sz = l >> 2, h = 0; h < 2; ++h, sz += 4)
    win_flush_run(c + sz * kWinZ, kWinY, grad, gx + clamp_index(w.lo[2] + ((sz - w.lo[2]) & 7), v.nz) * nxy, w.lo[1], v.ny, nx);
}

// Move the origin of the lanes' windows along one axis to `to` (uniform over a
// group), flushing what drops out.
template <int A>
__device__ inline void win_move_axis(GradWindow &w, float *grad, const VolConst &v, int to) {
  constexpr int N = A == 0 ? kWinX : kWin;
  const int at = w.lo[A], p1 = to > at ? min(to, at + N) : at + N;
  for (int p = to > at ? at : max(to + N, at); p < p1; p += A == 0 ? 4 : 1) {
    if constexpr (A == 0)
      win_flush_quad(w, grad, v, p);
    else
      win_flush_plane<A>(w, grad, v, p);
  }
  w.lo[A] = to;
  if constexpr (A == 0) {
    const int s = w.sx + (to - at);
    w.sx = s >= 0 && s < N ? s : (s >= N && s < 2 * N ? s - N : (s < 0 && s >= -N ? s + N : 0));
  }
}

// Empty every group's window (the whole wavefront calls it).
__device__ inline void win_flush(GradWindow &w, float *grad, const VolConst &v) {
  if (w.valid) win_move_axis<1>(w, grad, v, w.lo[1] + kWin);  // (every plane in y)
  w.valid = false;
}

// Place the windows over the stencil bases b of the lanes in `staged`; true
// for the lanes of groups whose stencils fit a window.
__device__ inline bool win_place(GradWindow &w, float *grad, const VolConst &v, bool staged, const int b[3]) {
  const bool in = w.valid && (uint32_t)(b[0] - w.lo[0]) <= (uint32_t)kSpreadX &&
                  (uint32_t)(b[1] - w.lo[1]) <= (uint32_t)kSpread && (uint32_t)(b[2] - w.lo[2]) <= (uint32_t)kSpread;
  if (__ballot(staged && !in) == 0ull) return true;
  int mn[3], mx[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    mn[a] = row_min_i32(staged ? b[a] : 0x7fffffff);
    mx[a] = -row_min_i32(staged ? -b[a] : 0x7fffffff);
  }
  if (mn[0] == 0x7fffffff) return true;  // a group without a sample
  const int x4 = mn[0] & ~3;
  if (mx[0] - x4 > kSpreadX || mx[1] - mn[1] > kSpread || mx[2] - mn[2] > kSpread) return false;
  if (!w.valid) {
    w.lo[0] = x4;
    w.lo[1] = mn[1];
    w.lo[2] = mn[2];
    w.sx = 0;
    w.valid = true;
    return true;
  }
  // Once a group's stencils leave its window along an axis, every group moves
  // along it, as far ahead in its rays' direction as its stencils allow: the
  // wavefront flushes all groups' planes together, and less often.
  auto target = [&](int a, int spread, int low, int high) {  // origins that start at mn, that end with mx
    const bool past = mx[a] > w.lo[a] + spread, before = mn[a] < w.lo[a];
    const bool move = __ballot(past || before) != 0ull;
    return !move ? w.lo[a] : (past || (!before && (w.ahead >> a & 1)) ? low : high);
  };
  const int tx = target(0, kSpreadX, x4, min((mx[0] - kSpreadX + 3) & ~3, x4));
  const int ty = target(1, kSpread, mn[1], mx[1] - kSpread), tz = target(2, kSpread, mn[2], mx[2] - kSpread);
  win_move_axis<0>(w, grad, v, tx);
  win_move_axis<1>(w, grad, v, ty);
  win_move_axis<2>(w, grad, v, tz);
  return true;
}

// One round: the sample of lane R of every group.  The broadcasts ride in the
// adds and multiply-adds as DPP operands, which the compiler does not fold for
// row_newbcast into fmac (20 VALU instructions a round instead of 10).  s_nop 1:
// the two wait states between a VALU write and a DPP read of the register.
template <int R, int STEP, int N, int I = 0>
__device__ inline void win_round(const float prod[N], const float wy[4], int x, int z, const int ysel[4], int a, int c) {
  uint32_t c0, c1, c2, c3;
  // c0 = x slot of tap a in bytes (x + a, less 48 when past the window), c1 = z
  // slot of tap c, c3 = their offset, then the four y taps' addresses
  asm("s_nop 1\n\t"
      "v_add_u32_dpp %0, %4, %5 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %6, %7 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32 %2, %12, %0\n\t"
      "v_and_b32 %1, 7, %1\n\t"
      "v_min_u32 %0, %0, %2\n\t"
      "v_mad_u32_u24 %3, %1, 48, %0\n\t"
      "v_add_u32_dpp %0, %8, %3 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %9, %3 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %2, %10, %3 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %3, %11, %3 row_newbcast:%c13 row_mask:0xf bank_mask:0xf"
      : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3)
      : "v"(x), "v"(a), "v"(z), "v"(c), "v"(ysel[0]), "v"(ysel[1]), "v"(ysel[2]), "v"(ysel[3]), "i"(-4 * kWinX), "i"(R));
  float v0 = *lds_at(c0), v1 = *lds_at(c1), v2 = *lds_at(c2), v3 = *lds_at(c3);
  asm("s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %4, %8 row_newbcast:%c9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %5, %8 row_newbcast:%c9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %6, %8 row_newbcast:%c9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %7, %8 row_newbcast:%c9 row_mask:0xf bank_mask:0xf"
      : "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3)
      : "v"(wy[0]), "v"(wy[1]), "v"(wy[2]), "v"(wy[3]), "v"(prod[I]), "i"(R));
  *lds_at(c0) = v0;
  *lds_at(c1) = v1;
  *lds_at(c2) = v2;
  *lds_at(c3) = v3;
  if constexpr (I < N - 1) win_round<R + STEP, STEP, N, I + 1>(prod, wy, x, z, ysel, a, c);
}

// The samples of lanes R, R + STEP, .., R + (N - 1) STEP of every group (N = 2,
// 4 or 8).
template <int R, int STEP, int N>
__device__ inline bool win_in_batch() {
  const int l = (int)(threadIdx.x % 16);
  return STEP == 1 ? l / N == R / N : l % STEP == R;
}

template <int R, int STEP, int N>
__device__ inline void win_batch(const GradWindow &w, const VolConst &v, bool staged, const int b[3], const Stencil &st, float dv) {
  const int l = (int)(threadIdx.x % 16);
  if (win_in_batch<R, STEP, N>()) {
    const float d = staged ? dv : 0.0f;
    lds_float *mine = w.prod + (STEP == 1 ? l % N : l / STEP) * kProdLane;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float wz = d * st.wz[q];
      const f32x4 t = {wz * st.wx[0], wz * st.wx[1], wz * st.wx[2], wz * st.wx[3]};
      *(lds_f32x4 *)(mine + 4 * q) = t;
    }
  }
  // this sample's slots (of any cell of the window when it is not staged)
  int x = staged ? b[0] - w.lo[0] + w.sx : 0;
  x = 4 * (x >= kWinX ? x - kWinX : x);
  int ysel[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) ysel[i] = (int)lds_address(w.cells) + ((b[1] + i) & 7) * (4 * kWinY);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  float prod[N];
#pragma unroll
  for (int r = 0; r < N; ++r) prod[r] = w.prod[r * kProdLane + l];
  win_round<R, STEP, N>(prod, st.wy, x, b[2] & 7, ysel, 4 * (l & 3), l >> 2);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// How an instantiation adds up the grid gradient.  Windows cover a whole step,
// or are placed for N consecutive lanes at a time (samples of one ray, G = 16), or
// for the rays' first samples, then their second ones, and so on.
enum Scatter { kWinStep = 0, kWinRay = 1, kWinSample = 2, kWaveBox = 3, kNoGrid = 4 };

// Add dv times the stencil weights of every lane in `staged` (the whole
// wavefront calls it).  A group spread wider than a window adds its taps to
// global memory.
template <int G, int MODE, int N>
__device__ inline void win_add(GradWindow &w, float *grad, const VolConst &v, bool staged, const Stencil &st, float dv) {
  const int b[3] = {st.ix - 1, st.iy - 1, st.iz - 1};
  if constexpr (MODE == kWinStep) {
    const bool fits = win_place(w, grad, v, staged, b);
    if (staged && !fits) scatter_taps(grad, v, st, dv);
    win_batch<0, 1, 8>(w, v, staged && fits, b, st, dv);
    win_batch<8, 1, 8>(w, v, staged && fits, b, st, dv);
  } else {
    auto batch = [&](auto H_) {
      constexpr int STEP = MODE == kWinRay ? 1 : G, R = decltype(H_)::value * (MODE == kWinRay ? N : 1);
      const bool here = staged && win_in_batch<R, STEP, N>();
      if (__ballot(here) == 0ull) return;
      const bool fits = win_place(w, grad, v, here, b);
      if (here && !fits) scatter_taps(grad, v, st, dv);
      win_batch<R, STEP, N>(w, v, here && fits, b, st, dv);
    };
    for_each_index<16 / N>(batch);
  }
}

// ---------------------------------------------------------------------------
// Gradient box, for long steps: each wavefront accumulates its grid gradient in a
// 14 x 14 x 14 box of LDS placed over the slab its lanes are sampling; when a
// step's stencils leave the box, the box is flushed to global memory (one atomic
// per touched voxel) and placed anew.  Samples two voxels and more apart along
// their rays share cells with their neighbours' only, so a window of 16 lanes
// flushes nearly all it gathers, once per window; the box holds what 32 rays
// share.  Steps whose stencils spread wider than the box add their taps to
// global memory.
// ---------------------------------------------------------------------------
constexpr int kBox = 14;   // box extent per axis
constexpr int kBoxY = 16;  // y stride
// z stride: with y stride 16 and z stride 228 the 64 taps a + 16 b + 228 c
// (a, b, c < 4) of one stencil fall in 64 distinct LDS banks
constexpr int kBoxZ = kBoxY * kBox + 4;
constexpr int kBoxCells = kBox * kBoxZ;
constexpr int kRec = 16;  // dwords per staged scatter record
constexpr int kBoxFloats = kBoxCells + kWaveSize * kRec;  // of one wavefront
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i32x4 lds_i32x4;

struct GradBox {
  lds_float *cells;  // this wavefront's cells, [z][y][x], zero outside use; nullptr: no box
  lds_float *recs;   // this wavefront's staged scatter records, kRec dwords per slot
  int ox, oy, oz;
  bool valid;
};

__device__ inline void box_flush(GradBox &b, float *grad, const VolConst &v) {
  if (!b.valid) return;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int lane = threadIdx.x % kWaveSize;
  for (int i = lane; i < kBox * kBox * kBox; i += kWaveSize) {
    const int cx = i % kBox, cy = (i / kBox) % kBox, cz = i / (kBox * kBox);
    const int cell = cz * kBoxZ + cy * kBoxY + cx;
    const float val = b.cells[cell];
    if (val != 0.0f) {
      const int x = b.ox + cx, y = b.oy + cy, z = b.oz + cz;
      if (x < v.nx && y < v.ny && z < v.nz)
        unsafeAtomicAdd(grad + ((uint32_t)z * (uint32_t)v.ny + (uint32_t)y) * (uint32_t)v.nx + (uint32_t)x, val);
      b.cells[cell] = 0.0f;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  b.valid = false;
}

// Wavefront-wide: make the box cover every clamped stencil of this step's
// sampling lanes, if they fit.
__device__ inline void box_prepare(GradBox &b, float *grad, const VolConst &v, const Ray &r, bool want, float px,
                                   float py, float pz) {
  int lo[3] = {0x7fffffff, 0x7fffffff, 0x7fffffff}, hi[3] = {-1, -1, -1};
  const int n[3] = {v.nx, v.ny, v.nz};
  if (want) {
    const float p[3] = {px, py, pz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int f = (int)floorf(p[a]);
      lo[a] = min(max(f - 1, 0), n[a] - 1);
      hi[a] = min(max(f + 2, 0), n[a] - 1);
    }
  }
  const int o[3] = {b.ox, b.oy, b.oz};
  bool inside = true;
  if (want)
#pragma unroll
    for (int a = 0; a < 3; ++a) inside = inside && lo[a] >= o[a] && hi[a] < o[a] + kBox;
  if (b.valid && __ballot(!inside) == 0ull) return;
  box_flush(b, grad, v);
  int mn[3], mx[3];
  bool fits = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    mn[a] = wave_min_i32(lo[a]);
    mx[a] = wave_max_i32(hi[a]);
    fits = fits && (mx[a] - mn[a] < kBox);
  }
  if (!fits) return;  // this step scatters to global memory
  // extend the box along the marching direction of the first sampling lane
  const unsigned long long wm = __ballot(want);
  const int first = __ffsll((long long)wm) - 1;
  int org[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float da = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, r.d[a]), first));
    org[a] = max(da >= 0.0f ? mn[a] : mx[a] - kBox + 1, 0);
  }
  b.ox = __builtin_amdgcn_readfirstlane(org[0]);
  b.oy = __builtin_amdgcn_readfirstlane(org[1]);
  b.oz = __builtin_amdgcn_readfirstlane(org[2]);
  b.valid = true;
}

// A lane whose stencil is interior stages its scatter record (x, y, z weights
// with dv folded into the z weights, the box cell of tap (0, 0, 0) and its
// coordinates); the wavefront then applies the staged records with the lanes
// transposed onto the 64 taps (box_apply).  Clamped stencils, whose taps can
// coincide, add their taps with LDS atomics right away.
__device__ inline bool box_stage(GradBox &b, const VolConst &v, const Stencil &st, float dv) {
  const bool inner = (st.ix >= 1) & (st.ix + 2 <= v.nx - 1) & (st.iy >= 1) & (st.iy + 2 <= v.ny - 1) &
                     (st.iz >= 1) & (st.iz + 2 <= v.nz - 1);
  if (inner) {
    // records are packed in lane order: this lane's slot is its rank among
    // the staging lanes (all of which are active here together)
    const unsigned long long act = __ballot(1);
    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0u));
    lds_float *rec = b.recs + rank * kRec;
    const f32x4 wx = {st.wx[0], st.wx[1], st.wx[2], st.wx[3]};
    const f32x4 wy = {st.wy[0], st.wy[1], st.wy[2], st.wy[3]};
    const f32x4 wz = {dv * st.wz[0], dv * st.wz[1], dv * st.wz[2], dv * st.wz[3]};
    *(lds_f32x4 *)(rec + 0) = wx;
    *(lds_f32x4 *)(rec + 4) = wy;
    *(lds_f32x4 *)(rec + 8) = wz;
    // box coordinates of tap (0, 0, 0): its cell, and two packings used to
    // find where two records' stencils overlap
    const int x = st.ix - 1 - b.ox, y = st.iy - 1 - b.oy, z = st.iz - 1 - b.oz;
    const i32x4 m = {z * kBoxZ + y * kBoxY + x, x + 16 * y + 256 * z, 4 * (x + 4 * y + 16 * z), 0};
    *(lds_i32x4 *)(rec + 12) = m;
    return true;
  }
  int xs[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) xs[a] = min(max(st.ix - 1 + a, 0), v.nx - 1) - b.ox;
  for (int c = 0; c < 4; ++c) {
    const int z = min(max(st.iz - 1 + c, 0), v.nz - 1) - b.oz;
    const float wc = dv * st.wz[c];
    for (int bb = 0; bb < 4; ++bb) {
      const int y = min(max(st.iy - 1 + bb, 0), v.ny - 1) - b.oy;
      const float wb = wc * st.wy[bb];
#pragma unroll
      for (int a = 0; a < 4; ++a)
        __hip_atomic_fetch_add(b.cells + z * kBoxZ + y * kBoxY + xs[a], wb * st.wx[a], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  return false;
}

// Wavefront-wide: apply the records of the lanes in `staged` (packed in slots
// 0 .. n-1 by box_stage).  For one record the 64 lanes update 64 distinct
// cells in 64 distinct banks, so a plain read-add-write is exact.  Records are
// applied two at a time with one LDS round trip: both cells are read before
// either is written, and where the second record's tap lands on a cell of the
// first record's stencil, the lane adds the first record's weight for that cell,
// fetched from the lane that owns it with a cross-lane permute; the writes go out
// in record order, so a cell shared by the two ends up with both contributions.
// The next pair's record words are read before this pair's cells are written
// (records never alias cells).  An odd last record is applied on its own.
__device__ inline void box_apply(GradBox &b, unsigned long long staged) {
  if (staged == 0ull) return;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int l = threadIdx.x % kWaveSize;
  const int ta = l & 3, tb = (l >> 2) & 3, tc = l >> 4;
  const int off = tc * kBoxZ + tb * kBoxY + ta;
  // tap coordinates biased by 4 in 4-bit fields: adding another record's
  // offset (x + 16 y + 256 z) leaves every field in [4, 7] exactly when the
  // shifted tap is inside that record's stencil
  const int tp = (ta + 4) + 16 * (tb + 4) + 256 * (tc + 4);
  const int l4 = 4 * l;
  const int n = __popcll(staged);
  struct Pair {
    float x[2], y[2], z[2];  // this lane's tap weights, not yet multiplied
    int cell[2], P[2], Q4[2];
  };
  auto load_pair = [&](int i, Pair &q) {  // records i and i + 1 (adjacent slots)
    const lds_float *r0 = b.recs + i * kRec, *r1 = r0 + kRec;
    const i32x4 m0 = *(const lds_i32x4 *)(r0 + 12), m1 = *(const lds_i32x4 *)(r1 + 12);
    q.x[0] = r0[ta];
    q.y[0] = r0[4 + tb];
    q.z[0] = r0[8 + tc];
    q.x[1] = r1[ta];
    q.y[1] = r1[4 + tb];
    q.z[1] = r1[8 + tc];
    q.cell[0] = m0.x + off;
    q.P[0] = m0.y;
    q.Q4[0] = m0.z;
    q.cell[1] = m1.x + off;
    q.P[1] = m1.y;
    q.Q4[1] = m1.z;
  };
  int i = 0;
  if (n >= 2) {
    Pair cur;
    load_pair(0, cur);
    for (;;) {
      const float w0 = cur.x[0] * cur.y[0] * cur.z[0];
      const float w1 = cur.x[1] * cur.y[1] * cur.z[1];
      // the first record's weight at this lane's tap of the second record
      const float c = __builtin_bit_cast(
          float, __builtin_amdgcn_ds_bpermute(l4 + cur.Q4[1] - cur.Q4[0], __builtin_bit_cast(int, w0)));
      const float v0 = b.cells[cur.cell[0]];
      float v1 = b.cells[cur.cell[1]];
      const bool more = i + 3 < n;
      Pair nxt;
      if (more) load_pair(i + 2, nxt);
      const int t = tp + cur.P[1] - cur.P[0];
      v1 += (t & 0xCCC) == 0x444 ? c : 0.0f;
      b.cells[cur.cell[0]] = v0 + w0;
      b.cells[cur.cell[1]] = v1 + w1;
      i += 2;
      if (!more) break;
      cur = nxt;
    }
  }
  if (i < n) {  // an odd last record
    const lds_float *r = b.recs + i * kRec;
    const float w = r[ta] * r[4 + tb] * r[8 + tc];
    const int cell = (*(const lds_i32x4 *)(r + 12)).x + off;
    b.cells[cell] += w;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The adjoint marches each ray with a group of G lanes (see walk_group): every
// lane recomputes its own samples, the group's chain gives each lane T_k a_k,
// T_{k+1} and C_{<=k} of its sample, and the lane applies that sample's
// adjoint.
template <int G, int MODE, int N, int DT>
__device__ inline void march_backward(const VolConst &v, const TfShared &s, lds_double *sgtf, GradWindow &win, GradBox &box,
                                      const TfConst &tf, const MarchConst &mc, const Ray &r,
                                      __amdgpu_buffer_rsrc_t rs, float4 g, float4 fin, float *grad_vol) {
  const float sl2 = mc.step * 1.4426950408889634f;
  const float Tend = 1.0f - fin.w;
  // TF-gradient contributions are summed in registers for the two nodes of
  // the current TF segment (ga[0..3]: node cj, ga[4..7]: node cj + 1).  When
  // the segment moves by one node, the shared node's sums stay in registers
  // and only the node left behind is added to LDS; otherwise both are.  (Every
  // sample added to LDS at once: 140 -> 144 ms and 6.6 -> 8.5 ms on the cases
  // above, lanes of a ray then adding to one word in the same instruction.)
  int cj = -1;
  float ga[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  auto add_node = [&](int node, const float *val) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (val[i] != 0.0f)
        __hip_atomic_fetch_add(sgtf + i * tf.K + node, (double)val[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto flush_tf = [&]() {
    if (cj >= 0) {
      add_node(cj, ga);
      add_node(cj + 1, ga + 4);
    }
  };
  auto move_tf = [&](int j) {
    const bool up = j == cj + 1, down = j == cj - 1;
    if (cj >= 0) {
      // left behind: node cj when moving up, node cj + 1 when moving down
      float lv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) lv[i] = down ? ga[4 + i] : ga[i];
      add_node(down ? cj + 1 : cj, lv);
      if (!up && !down) add_node(cj + 1, ga + 4);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float keep = up ? ga[4 + i] : (down ? ga[i] : 0.0f);
      ga[i] = down ? 0.0f : keep;
      ga[4 + i] = down ? keep : 0.0f;
    }
    cj = j;
  };
  bool staged = false;  // this lane's sample scatters sdv
  float sdv = 0.0f;
  auto prep = [&](bool want, float px, float py, float pz) {
    if constexpr (MODE == kWaveBox)
      if (grad_vol && box.cells) box_prepare(box, grad_vol, v, r, want, px, py, pz);
  };
  // the taps of this lane's next lattice point are loaded while this one is
  // processed (in the adjoint every lattice point of a ray is usually visited)
  TapPrefetch<DT> pf;
  pf.ix = INT_MIN;
  float sx = 0.0f, sy = 0.0f, sz = 0.0f;  // this lane's sample: its position
  Classified cq;                          // and classification, kept for its adjoint
  auto eval = [&](int k, float px, float py, float pz) -> ChainSample {
    sx = px;
    sy = py;
    sz = pz;
    const Stencil st = make_stencil(px, py, pz);
    const float val = reconstruct_prefetched<DT>(pf, rs, v, st);
    if (k + G < r.k0 + r.ns) {
      float qx, qy, qz;
      lattice_point(r, mc.step, k + G, qx, qy, qz);
      prefetch_taps<DT>(pf, rs, v, (int)floorf(qx), (int)floorf(qy), (int)floorf(qz));
    }
    cq = classify(s, tf.K, tf.v0, tf.scale, val);
    return ChainSample{cq.c.x, cq.c.y, cq.c.z, transmit(cq.c.w, sl2)};
  };
  // TF gradient of the dsig-only adjoint of one sample with classification q
  // (its colour gradient is zero: T_k a_k = 0), n identical samples at once
  auto tf_sigma = [&](const Classified &q, float dsig, float n) {
    if (q.j != cj) move_tf(q.j);
    const float d = n * dsig;
    ga[3] = fmaf(1.0f - q.w, d, ga[3]);
    ga[7] = fmaf(q.w, d, ga[7]);
  };
  // n samples of a constant empty block (extinction 0, so a = 0 and the ray's
  // state is unchanged): only dsig is non-zero, the same for all of them
  auto flat = [&](int n, const ChainState &o, float value) {
    if (!sgtf) return;
    const Classified fq = classify(s, tf.K, tf.v0, tf.scale, value);
    float acc = g.w * Tend;
    acc = fmaf(g.x, o.T * fq.c.x - (fin.x - o.C0), acc);
    acc = fmaf(g.y, o.T * fq.c.y - (fin.y - o.C1), acc);
    acc = fmaf(g.z, o.T * fq.c.z - (fin.z - o.C2), acc);
    tf_sigma(fq, mc.step * acc, (float)n);
  };
  // adjoint of this lane's sample k, given T_k a_k, T_{k+1} and C_{<=k}
  auto take = [&](bool mine, const ChainState &o) {
    if (!mine) return;
    const float ta = o.ta, T = o.T;
    float dc0 = g.x * ta, dc1 = g.y * ta, dc2 = g.z * ta;
    float acc = g.w * Tend;
    acc = fmaf(g.x, T * cq.c.x - (fin.x - o.C0), acc);
    acc = fmaf(g.y, T * cq.c.y - (fin.y - o.C1), acc);
    acc = fmaf(g.z, T * cq.c.z - (fin.z - o.C2), acc);
    float dsig = mc.step * acc;
    if (sgtf) {
      if (cq.j != cj) move_tf(cq.j);
      float w1 = cq.w, w0 = 1.0f - cq.w;
      ga[0] = fmaf(w0, dc0, ga[0]);
      ga[1] = fmaf(w0, dc1, ga[1]);
      ga[2] = fmaf(w0, dc2, ga[2]);
      ga[3] = fmaf(w0, dsig, ga[3]);
      ga[4] = fmaf(w1, dc0, ga[4]);
      ga[5] = fmaf(w1, dc1, ga[5]);
      ga[6] = fmaf(w1, dc2, ga[6]);
      ga[7] = fmaf(w1, dsig, ga[7]);
    }
    if (MODE != kNoGrid && grad_vol && !cq.clamped) {
      float4 a = s.node[cq.j], b = s.node[cq.j + 1];
      float dv = dc0 * (b.x - a.x);
      dv = fmaf(dc1, b.y - a.y, dv);
      dv = fmaf(dc2, b.z - a.z, dv);
      dv = fmaf(dsig, b.w - a.w, dv);
      dv *= tf.scale;
      if constexpr (MODE == kWaveBox) {
        if (dv != 0.0f) {
          const Stencil st = make_stencil(sx, sy, sz);
          if (box.valid)
            staged = box_stage(box, v, st, dv);
          else
            scatter_taps(grad_vol, v, st, dv);
        }
      } else {
        staged = dv != 0.0f;
        sdv = dv;
      }
    }
  };
  auto post = [&]() {
    if constexpr (MODE == kNoGrid) return;
    if (!grad_vol || __ballot(staged) == 0ull) return;
    if constexpr (MODE == kWaveBox) {
      box_apply(box, __ballot(staged));
      staged = false;
      return;
    }
    const Stencil st = make_stencil(sx, sy, sz);  // (recomputed: fewer registers across the chain)
    if constexpr (MODE < kWaveBox) {
      if (win.cells)
        win_add<G, MODE, N>(win, grad_vol, v, staged, st, sdv);
      else if (staged)
        scatter_taps(grad_vol, v, st, sdv);
    }
    staged = false;
  };
  win.ahead = __builtin_amdgcn_mov_dpp((r.d[0] >= 0.0f ? 1 : 0) | (r.d[1] >= 0.0f ? 2 : 0) | (r.d[2] >= 0.0f ? 4 : 0),
                                       0x150, 0xF, 0xF, true);  // the group's first ray's (row_newbcast:0)
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 1.0f);
  walk_group<G, true>(v, s, tf, mc, r, eval, prep, take, flat, post, acc);
  if (sgtf) flush_tf();
  if constexpr (MODE == kWaveBox) {
    if (grad_vol) box_flush(box, grad_vol, v);
  } else if constexpr (MODE != kNoGrid) {
    if (grad_vol) win_flush(win, grad_vol, v);
  }
}

// Pixel of this lane's ray in wavefront w of part `part` of a super-tile:
// a tile of 8x4 (G = 2), 4x4 (G = 4) or 4x1 (G = 16) rays per wavefront, with the
// rays of 16 consecutive lanes (one gradient window) in a 4x2, 2x2 or 1x1 block.
template <int G>
__device__ inline void bwd_pixel_of(int sx, int sy, int part, int w, int &col, int &row) {
  constexpr int TW = G <= 2 ? 8 : 4, TH = kWaveSize / G / TW, WX = kSuperEdge / TW;
  constexpr int BW = G == 16 ? 1 : (G == 4 ? 2 : 4), BH = 16 / G / BW;
  const int lane = (int)(threadIdx.x % kWaveSize), sub = lane / 16, ray = lane % 16 / G;
  col = sx * kSuperEdge + (w % WX) * TW + (sub % (TW / BW)) * BW + ray % BW;
  row = sy * kSuperEdge + part * (kSuperEdge / G) + (w / WX) * TH + (sub / (TW / BW)) * BH + ray / BW;
}

#ifdef VR_TIMELINE
__device__ unsigned long long g_timeline_bwd[kTimelineWaves * 4];
static int64_t g_timeline_bwd_records = 0;
#endif

// One wavefront item of the adjoint: wavefront w of workgroup item i.
template <int DT, int G, int MODE, int N>
__device__ inline void backward_wave_item(const BackwardArgs &a, const TfShared &s, lds_double *sgtf, GradWindow &win,
                                          GradBox &box, __amdgpu_buffer_rsrc_t rs, int64_t i, int w) {
#ifdef VR_TIMELINE
  const unsigned long long tl0 = __builtin_amdgcn_s_memrealtime();
#endif
  const RenderArgs &ra = a.r;
  int part;
  const SuperTile st = group_tile_of<G>(ra.order, i, ra.W, ra.H, ra.n_views, ra.chunk_edge, part);
  if (!st.valid) return;  // uniform over the wavefront
  int col, row;
  bwd_pixel_of<G>(st.sx, st.sy, part, w, col, row);
  // every lane enters the march (it steps the wavefront in unison); lanes
  // outside the image or without a gradient carry an empty ray
  Ray r;
  r.hit = false;
  r.ns = 0;
  r.k0 = 0;
  r.d[0] = r.d[1] = r.d[2] = 0.0f;
  float4 g = make_float4(0.0f, 0.0f, 0.0f, 0.0f), fin = g;
  if (col < ra.W && row < ra.H) {
    size_t pix = ((size_t)st.view * ra.H + row) * ra.W + col;
    g = reinterpret_cast<const float4 *>(a.grad_rgba)[pix];
    if (g.x != 0.0f || g.y != 0.0f || g.z != 0.0f || g.w != 0.0f) {
      r = setup_ray(ra.cams[st.view], col, row, ra.vol.nx, ra.vol.ny, ra.vol.nz, ra.mc.step);
      fin = reinterpret_cast<const float4 *>(a.out_rgba)[pix];
    }
  }
  march_backward<G, MODE, N, DT>(ra.vol, s, sgtf, win, box, ra.tf, ra.mc, r, rs, g, fin, a.grad_vol);
#ifdef VR_TIMELINE
  const int tx = (ra.W + kSuperEdge - 1) / kSuperEdge, ty = (ra.H + kSuperEdge - 1) / kSuperEdge;
  timeline_record(g_timeline_bwd, (size_t)i * kWavesPerWg + w, tl0, st.view * tx * ty + st.sy * tx + st.sx,
                  (threadIdx.x % G) == 0 ? (uint32_t)r.ns : 0u);
#endif
}

// LDS holds two workgroups per CU (two wavefronts per SIMD): 256 registers.
// Queued like the forward (one workgroup item per workgroup without queue
// counters); a workgroup's TF gradient stays in its LDS over all its items.
template <int DT, int G, int MODE, int N>
__global__ __launch_bounds__(kWgSize) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_render_bwd(
    const BackwardArgs args) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const BackwardArgs &a = kernarg<BackwardArgs>();
  const RenderArgs &ra = a.r;
  const int K = ra.tf.K;
  const uint32_t tf_bytes = tf_lds_bytes(K);
  lds_double *sgtf = a.grad_tf ? (lds_double *)(lds + tf_bytes) : nullptr;
  if (sgtf)
    for (int j = threadIdx.x; j < 4 * K; j += kWgSize) sgtf[j] = 0.0;
  GradWindow win;
  win.valid = false;
  win.sx = win.ahead = 0;
  win.lo[0] = win.lo[1] = win.lo[2] = 0;
  win.cells = nullptr;
  win.prod = nullptr;
  GradBox box;
  box.valid = false;
  box.ox = box.oy = box.oz = 0;
  box.cells = box.recs = nullptr;
  if (MODE == kWaveBox && a.grad_vol && a.use_box) {
    box.cells = (lds_float *)(lds + grid_lds_offset(K, a.grad_tf != nullptr)) + (threadIdx.x / kWaveSize) * kBoxFloats;
    box.recs = box.cells + kBoxCells;
    for (int i = threadIdx.x % kWaveSize; i < kBoxCells; i += kWaveSize) box.cells[i] = 0.0f;
  }
  if (MODE < kWaveBox && a.grad_vol && a.use_box) {
    lds_float *wins = (lds_float *)(lds + grid_lds_offset(K, a.grad_tf != nullptr));
    const int row = (int)(threadIdx.x % kWaveSize) / 16;
    wins += (threadIdx.x / kWaveSize) * (kWinFloats + kProdFloats);
    for (int i = threadIdx.x % kWaveSize; i < kWinFloats; i += kWaveSize) wins[i] = 0.0f;
    win.cells = wins + row * kWinCells;
    win.prod = wins + kWinFloats + row * kProdRow;
  }
  TfShared s = carve_tf(lds, K);
  const bool tf_ok = load_tf(s, ra.tf);  // ends with a barrier, which also orders the zeroing
  if (!tf_ok) {
    // uniform over the launch: every workgroup fills its share of the
    // gradients with NaN and nothing is accumulated
    const float q = __builtin_nanf("");
    const int64_t nvox = (int64_t)ra.vol.nx * ra.vol.ny * ra.vol.nz;
    if (a.grad_vol)
      for (int64_t i = (int64_t)blockIdx.x * kWgSize + threadIdx.x; i < nvox; i += (int64_t)gridDim.x * kWgSize)
        a.grad_vol[i] = q;
    if (a.grad_tf && blockIdx.x == 0)
      for (int j = threadIdx.x; j < 4 * K; j += kWgSize) a.grad_tf[j] = q;
    return;
  }
  __amdgpu_buffer_rsrc_t rs = make_rsrc(ra.vol.data, ra.vol.bytes);
  if (!ra.queue) {
    int part;
    if (!group_tile_of<G>(ra.order, blockIdx.x, ra.W, ra.H, ra.n_views, ra.chunk_edge, part).valid)
      return;  // uniform over the workgroup
    backward_wave_item<DT, G, MODE, N>(a, s, sgtf, win, box, rs, blockIdx.x, (int)(threadIdx.x / kWaveSize));
  } else {
    const int x = (int)(blockIdx.x % kXcds);
    int w = 0;
    int64_t i = 0;
    while (next_wave_item(ra.queue, (uint32_t)ra.queue_items, x, i, w))
      backward_wave_item<DT, G, MODE, N>(a, s, sgtf, win, box, rs, i, w);
  }
  if (sgtf) {
    __syncthreads();
    for (int j = threadIdx.x; j < 4 * K; j += kWgSize) {
      const float val = (float)sgtf[(j & 3) * K + (j >> 2)];
      if (val != 0.0f) unsafeAtomicAdd(a.grad_tf + j, val);
    }
  }
}

template <int G, int MODE, int N>
static hipError_t launch_bwd_as(const BackwardArgs &a0, hipStream_t s, bool pairs = false) {
  BackwardArgs a = a0;
  const RenderArgs &ra = a.r;
  int64_t grid = group_grid(render_grid(ra), G);
#ifdef VR_TIMELINE
  g_timeline_bwd_records = grid * (kWgSize / kWaveSize);
#endif
  uint32_t lds = tf_lds_bytes(ra.tf.K) + tf_grad_bytes(ra.tf.K, a.grad_tf != nullptr);
  constexpr uint32_t wave_floats = MODE == kNoGrid ? 0u : (MODE == kWaveBox ? kBoxFloats : kWinFloats + kProdFloats);
  const uint32_t with_grid = grid_lds_offset(ra.tf.K, a.grad_tf != nullptr) + kWavesPerWg * wave_floats * 4u;
  a.use_box = MODE != kNoGrid && a.grad_vol && with_grid <= max_lds_per_workgroup() ? 1 : 0;
  if (a.use_box) lds = with_grid;
  auto *k = ra.vol.dtype == kU16 ? &k_render_bwd<kU16, G, MODE, N> : (ra.vol.dtype == kI16 ? &k_render_bwd<kI16, G, MODE, N> : &k_render_bwd<kF32, G, MODE, N>);
  if constexpr (MODE == kNoGrid)
    if (pairs && ra.vol.nx % 2 == 0 && ra.vol.dtype != kF32)
      k = ra.vol.dtype == kU16 ? &k_render_bwd<kU16Pairs, G, MODE, N> : &k_render_bwd<kI16Pairs, G, MODE, N>;
  const void *fn = reinterpret_cast<const void *>(k);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  a.r.queue = nullptr;
  a.r.queue_items = 0;
  if (ra.order) {
    const int64_t resident = resident_workgroups(fn, lds);
    if (resident >= kXcds && resident < grid) {
      a.r.queue = reinterpret_cast<uint32_t *>(const_cast<int32_t *>(ra.order) + tile_order_count(ra));
      a.r.queue_items = (int32_t)(grid / kXcds * kWavesPerWg);
      grid = resident;
    }
  }
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kWgSize), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_render_backward(const BackwardArgs &a, hipStream_t s) {
  const RenderArgs &ra = a.r;
  if (ra.vol.dtype != kU16 && ra.vol.dtype != kI16 && ra.vol.dtype != kF32) return hipErrorInvalidValue;
  const RayField f = ray_field(ra);
  if (!a.grad_vol) {
    // a wavefront whose taps fill a few lines gains nothing from the pairs'
    // alignment (256x256x200 to 512^2, p = 0.11, step 0.5, two lanes: 2.59 ms by voxel,
    // 2.83 by pair, step 1: 1.70, 1.48; step 4, one lane: 0.37, 0.40)
    const int group = lanes_within(tf_adjoint_group(f, ra.mc.step), render_grid(ra));
    const bool pairs = group == 1 ? f.pitch >= 0.2 : f.pitch * ra.mc.step >= 0.1;
    switch (group) {
    case 16: return launch_bwd_as<16, kNoGrid, 1>(a, s, pairs);
    case 4: return launch_bwd_as<4, kNoGrid, 1>(a, s, pairs);
    case 1: return launch_bwd_as<1, kNoGrid, 1>(a, s, pairs);
    default: return launch_bwd_as<2, kNoGrid, 1>(a, s, pairs);
    }
  }
  Adjoint shape = adjoint_shape(f, ra.mc.step);
  if (shape == Adjoint::k1 && lanes_within(16, render_grid(ra)) < 16) shape = Adjoint::k2x2Sample;
  if (shape == Adjoint::k2x2Sample && lanes_within(4, render_grid(ra)) < 4) shape = Adjoint::k4x2Sample;
  switch (shape) {
  case Adjoint::k4x4: return launch_bwd_as<1, kWinStep, 8>(a, s);
  case Adjoint::k4x2Step: return launch_bwd_as<2, kWinStep, 8>(a, s);
  case Adjoint::k4x2Sample: return launch_bwd_as<2, kWinSample, 8>(a, s);
  case Adjoint::k2x2Sample: return launch_bwd_as<4, kWinSample, 4>(a, s);
  case Adjoint::k1: return launch_bwd_as<16, kWinRay, 4>(a, s);
  default: return launch_bwd_as<2, kWaveBox, 8>(a, s);
  }
}

#ifdef VR_TIMELINE
int64_t timeline_copy_bwd(unsigned long long *host, int64_t max) {
  const int64_t n = std::min<int64_t>(std::min<int64_t>(g_timeline_bwd_records, kTimelineWaves), max);
  if (hipDeviceSynchronize() != hipSuccess) return -1;
  if (n > 0 && hipMemcpyFromSymbol(host, HIP_SYMBOL(g_timeline_bwd), (size_t)n * 4 * sizeof(unsigned long long)) != hipSuccess)
    return -1;
  return g_timeline_bwd_records;
}
#endif

}  // namespace vr
