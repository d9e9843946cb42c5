// frame_prep.hip -- what a render needs before its first ray (gfx950): the
// blocks' occupancy under the TF, the radii of empty cubes around them, and the
// order of its workgroups.
#include <algorithm>

#include "vr_internal.h"

namespace vr {

// ---------------------------------------------------------------------------
// Centre-out workgroup order: a counting sort of the super-tiles by their
// distance to the projected volume centre (half-tile rings) and, within a
// ring, by angle around the centre (32 sectors), in one workgroup.  Item i of
// the order runs on XCD i mod 8, so the angular order spreads every XCD's
// tiles around each ring: an XCD does not inherit one side of the volume (in
// raster order the two sides of a ring alternate, and the XCDs of one parity
// took one side: 7.5 % more work on four of them for the C1 frame).  Items of
// one (ring, sector) key come in any order; the image does not depend on the
// order.
// ---------------------------------------------------------------------------
constexpr int kOrderRings = 256;
constexpr int kOrderSectors = 32;
constexpr int kOrderKeys = kOrderRings * kOrderSectors;
constexpr int kPrepThreads = 1024;
constexpr int kKeysPerThread = kOrderKeys / kPrepThreads;
// LDS of the order: the keys' counts and the wavefronts' totals
constexpr uint32_t kOrderLdsBytes = (kOrderKeys + kPrepThreads / kWaveSize) * 4;

struct OrderArgs {
  float cx[kMaxCamsPerLaunch], cy[kMaxCamsPerLaunch];  // centre, in super-tile units
  int32_t tx, ty, n_views;
};

__device__ inline int order_key(const OrderArgs &o, int q) {
  const int per = o.tx * o.ty, v = q / per, t = q % per;
  const float dx = (float)(t % o.tx) - o.cx[v], dy = (float)(t / o.tx) - o.cy[v];
  const float d = sqrtf(fmaf(dx, dx, dy * dy)) * 2.0f;
  const int ring = d < (float)(kOrderRings - 1) ? (int)d : kOrderRings - 1;
  const float turn = atan2f(dy, dx) * 0.15915494309189535f + 0.5f;  // in [0, 1]
  const int sector = min(max((int)(turn * (float)kOrderSectors), 0), kOrderSectors - 1);
  return ring * kOrderSectors + sector;
}

// One workgroup of kPrepThreads threads, kOrderLdsBytes of LDS at `cnt`.
__device__ inline void tile_order(const OrderArgs &o, int32_t *order, int *cnt) {
  int *wsum = cnt + kOrderKeys;
  const int n = o.n_views * o.tx * o.ty;
  for (int i = threadIdx.x; i < kOrderKeys; i += kPrepThreads) cnt[i] = 0;
  for (int i = threadIdx.x; i < (int)kOrderQueueInts; i += kPrepThreads) order[n + i] = 0;  // queue counters
  __syncthreads();
  for (int q = threadIdx.x; q < n; q += kPrepThreads) atomicAdd(&cnt[order_key(o, q)], 1);
  __syncthreads();
  // exclusive prefix sum of the counts: each thread sums its run of keys, an
  // inclusive scan of those sums inside each wavefront, then the wavefront totals
  const int lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
  int run[kKeysPerThread], c = 0;
#pragma unroll
  for (int i = 0; i < kKeysPerThread; ++i) {
    run[i] = cnt[threadIdx.x * kKeysPerThread + i];
    c += run[i];
  }
  int x = c;
#pragma unroll
  for (int off = 1; off < kWaveSize; off <<= 1) {
    const int y = __shfl_up(x, off, kWaveSize);
    if (lane >= off) x += y;
  }
  if (lane == kWaveSize - 1) wsum[wave] = x;
  __syncthreads();
  int before = x - c;
  for (int w = 0; w < wave; ++w) before += wsum[w];
#pragma unroll
  for (int i = 0; i < kKeysPerThread; ++i) {
    cnt[threadIdx.x * kKeysPerThread + i] = before;
    before += run[i];
  }
  __syncthreads();
  for (int q = threadIdx.x; q < n; q += kPrepThreads) order[atomicAdd(&cnt[order_key(o, q)], 1)] = q;
}

__global__ __launch_bounds__(kPrepThreads) void k_tile_order(const OrderArgs o, int32_t *order) {
  __shared__ int cnt[kOrderLdsBytes / 4];
  tile_order(o, order, cnt);
}

// ---------------------------------------------------------------------------
// Both planes in one launch: the occupancy bits (plane 0, as k_occupancy_bits)
// and the radius plane after them: 2 bits per block (16 blocks a word), for
// an empty block b the largest r <= kEmptyRadiusMax such that every block
// within Chebyshev distance r of b is empty (outside the grid counts as
// empty), 0 for occupied blocks.  The blocks around a workgroup's
// kPrepThreads consecutive blocks lie within empty_reach bit positions of
// them: the workgroup decides the occupancy of that window itself (from
// min/max and the TF in LDS), writes plane 0 for its own blocks, and reads
// each x-row of a neighbourhood as one bit field of at most 2R + 1 bits.
// Workgroups of 1024 threads: the window (three planes of blocks on either
// side) is shared by four times the blocks of a 256-thread workgroup.
//
// What bounds it: latency, a few dozen workgroups each walking one chain (TF,
// ranges, decisions, neighbourhoods).  The ranges of kPrepBatch blocks per lane
// are in flight together, the first of them while the TF is loaded, and the 49
// rows of a neighbourhood are read without a branch.
//
// The workgroup order of the frame, when asked for, is one more workgroup of
// the same launch (the last): the two are independent.  A range loaded and
// decided after the other and two launches took 18 + 9 us before a frame of
// 512x512x400 in 16-voxel blocks (25600 of them), 10.4 us now, and 10.8 + 4 us
// before one of 97x81x73 (210 blocks), 5.1 us now (the frame to 128x96: 70 -> 62 us).
// ---------------------------------------------------------------------------
constexpr int kPrepBatch = 8;
__host__ __device__ inline int64_t empty_reach(const VolConst &v) {
  return kEmptyRadiusMax * (1 + (int64_t)v.nbx + (int64_t)v.nbx * v.nby);
}
__host__ __device__ inline int64_t empty_window_words(const VolConst &v) {
  return (kPrepThreads + 2 * empty_reach(v)) / 32 + 2;
}
__host__ __device__ inline uint32_t planes_lds_bytes(const VolConst &v, int K) {
  return ((tf_lds_bytes(K) + 15u) & ~15u) + (uint32_t)empty_window_words(v) * 4u;
}

// Bits 0..15 of x moved to the even positions 0, 2, .., 30.
__device__ inline uint32_t spread16(uint32_t x) {
  x &= 0xffffu;
  x = (x | (x << 8)) & 0x00ff00ffu;
  x = (x | (x << 4)) & 0x0f0f0f0fu;
  x = (x | (x << 2)) & 0x33333333u;
  x = (x | (x << 1)) & 0x55555555u;
  return x;
}

__global__ __launch_bounds__(kPrepThreads) void k_occupancy_planes(const VolConst v, const TfConst tf, uint32_t *bits,
                                                                   const OrderArgs o, int32_t *order) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  if (order && blockIdx.x == gridDim.x - 1) {  // uniform over the workgroup
    tile_order(o, order, reinterpret_cast<int *>(lds));
    return;
  }
  TfShared s = carve_tf(lds, tf.K);
  uint32_t *win = reinterpret_cast<uint32_t *>(lds + ((tf_lds_bytes(tf.K) + 15u) & ~15u));
  const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  const int64_t words = (nb + 31) / 32;
  const int64_t b0 = (int64_t)blockIdx.x * kPrepThreads;
  const int64_t w0 = max(b0 - empty_reach(v), (int64_t)0) >> 5;
  const int nw = (int)empty_window_words(v);
  // window occupancy: each wavefront decides 64 blocks (two words) at a time
  const int lane = threadIdx.x % kWaveSize, wave = threadIdx.x / kWaveSize;
  constexpr int kStride = 2 * (kPrepThreads / kWaveSize);  // window words between a wavefront's decisions
  float2 mm[kPrepBatch];
  auto fetch = [&](int j0) {
#pragma unroll
    for (int i = 0; i < kPrepBatch; ++i) {
      const int j = j0 + i * kStride;
      const int64_t q = 32 * (w0 + j) + lane;
      if (j < nw && q < nb) mm[i] = v.minmax[q];
    }
  };
  fetch(2 * wave);
  load_tf<kPrepThreads>(s, tf);  // ends with a barrier
  for (int j0 = 2 * wave; j0 < nw; j0 += kPrepBatch * kStride) {
    if (j0 != 2 * wave) fetch(j0);
#pragma unroll
    for (int i = 0; i < kPrepBatch; ++i) {
      const int j = j0 + i * kStride;
      if (j >= nw) break;  // uniform over the wavefront
      const bool in = 32 * (w0 + j) + lane < nb;
      const unsigned long long m = __ballot(in && range_occupied(s, tf.K, tf.v0, tf.scale, mm[i].x, mm[i].y));
      if (lane == 0) win[j] = (uint32_t)m;
      if (lane == 32 && j + 1 < nw) win[j + 1] = (uint32_t)(m >> 32);
    }
  }
  __syncthreads();
  if (threadIdx.x < kPrepThreads / 32) {  // plane 0 of this workgroup's blocks
    const int64_t w = (b0 >> 5) + threadIdx.x;
    if (w < words) bits[w] = win[w - w0];
  }
  const int64_t b = b0 + threadIdx.x;
  int rad = 0;
  if (b < nb) {
    const int bq = (int)b, nxy = v.nbx * v.nby;
    const int bz = bq / nxy, by = (bq - bz * nxy) / v.nbx, bx = bq - bz * nxy - by * v.nbx;
    constexpr int R = kEmptyRadiusMax;
    const int lx = max(bx - R, 0), hx = min(bx + R, v.nbx - 1), c = bx - lx;
    // ring[r]: blocks lx .. hx of the rows at distance max(|dy|, |dz|) = r, ored
    // together.  A row outside the grid is replaced by the nearest one inside,
    // which a ring of at most the same distance holds already.
    uint32_t ring[R + 1] = {0u};
#pragma unroll
    for (int dz = -R; dz <= R; ++dz) {
      const int z = min(max(bz + dz, 0), v.nbz - 1);
#pragma unroll
      for (int dy = -R; dy <= R; ++dy) {
        const int y = min(max(by + dy, 0), v.nby - 1);
        const int q = (int)(lx + (int64_t)v.nbx * (y + (int64_t)v.nby * z) - 32 * w0);
        const int w = q >> 5;
        const uint32_t lo = win[w], hi = win[min(w + 1, nw - 1)];  // (a field that crosses into w + 1 lies in the window)
        ring[max(abs(dy), abs(dz))] |= __builtin_amdgcn_alignbit(hi, lo, (uint32_t)q & 31u);
      }
    }
    // the largest r whose cube is empty; r = 0 is the block itself
    const uint32_t row = (1u << (hx - lx + 1)) - 1u;
    uint32_t field = 0u;
    int near = R + 1;  // smallest Chebyshev distance of an occupied block, capped at R + 1
#pragma unroll
    for (int r = 0; r <= R; ++r) {
      field |= ring[r] & row;
      const int lo = max(c - r, 0);
      const uint32_t within = ((1u << (c + r + 1)) - 1u) & ~((1u << lo) - 1u);
      if (near == R + 1 && (field & within)) near = r;
    }
    rad = near - 1 < 0 ? 0 : near - 1;
  }
  const unsigned long long lo = __ballot(rad & 1), hi = __ballot(rad & 2);
  const int64_t rw = words + (b >> 4);
  if ((lane & 15) == 0 && b < nb)
    bits[rw] = spread16((uint32_t)(lo >> lane)) | (spread16((uint32_t)(hi >> lane)) << 1);
}

bool occupancy_planes_fit(const VolConst &v, int K) { return planes_lds_bytes(v, K) <= max_lds_per_workgroup(); }

static OrderArgs order_args(const RenderArgs &a) {
  OrderArgs o{};
  o.tx = (a.W + kSuperEdge - 1) / kSuperEdge;
  o.ty = (a.H + kSuperEdge - 1) / kSuperEdge;
  o.n_views = a.n_views;
  const double p[3] = {0.5 * (a.vol.nx - 1), 0.5 * (a.vol.ny - 1), 0.5 * (a.vol.nz - 1)};
  for (int v = 0; v < a.n_views; ++v) {
    const CamConst &c = a.cams[v];
    double d[3], z = 0.0, x = 0.0, y = 0.0;
    for (int k = 0; k < 3; ++k) d[k] = p[k] - c.eye[k];
    for (int k = 0; k < 3; ++k) {
      z += d[k] * c.fwd[k];
      x += d[k] * c.right[k];
      y += d[k] * c.up[k];
    }
    double sx = 0.0, sy = 0.0;  // image centre when the volume centre does not project
    if (c.proj != 0) {
      if (z > 0.0) {
        sx = x / (z * c.th * ((double)c.W / (double)c.H));
        sy = y / (z * c.th);
      }
    } else {
      sx = c.hw > 0.0 ? x / c.hw : 0.0;
      sy = c.hh > 0.0 ? y / c.hh : 0.0;
    }
    const double col = (sx + 1.0) * 0.5 * c.W - 0.5, row = (1.0 - sy) * 0.5 * c.H - 0.5;
    o.cx[v] = (float)fmin(fmax((col + 0.5) / kSuperEdge - 0.5, -1e6), 1e6);
    o.cy[v] = (float)fmin(fmax((row + 0.5) / kSuperEdge - 0.5, -1e6), 1e6);
  }
  return o;
}

hipError_t launch_tile_order(const RenderArgs &a, int32_t *order, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_order, dim3(1), dim3(kPrepThreads), 0, s, order_args(a), order);
  return hipGetLastError();
}

int64_t tile_order_count(const RenderArgs &a) {
  return (int64_t)a.n_views * ((a.W + kSuperEdge - 1) / kSuperEdge) * ((a.H + kSuperEdge - 1) / kSuperEdge);
}

int32_t *alloc_tile_order(const RenderArgs &a, hipStream_t s) {
  int32_t *order = nullptr;
  if (hipMallocAsync((void **)&order, (size_t)(tile_order_count(a) + kOrderQueueInts) * sizeof(int32_t), s) != hipSuccess)
    return nullptr;
  return order;
}

int32_t *make_tile_order(const RenderArgs &a, hipStream_t s) {
  int32_t *order = alloc_tile_order(a, s);
  if (order && launch_tile_order(a, order, s) != hipSuccess) {
    (void)hipFreeAsync(order, s);
    return nullptr;
  }
  return order;
}

static hipError_t launch_planes(const VolConst &v, const TfConst &tf, uint32_t *bits, const OrderArgs &o, int32_t *order,
                                hipStream_t s) {
  if (!occupancy_planes_fit(v, tf.K)) return hipErrorInvalidValue;  // the caller leaps block by block
  const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  const uint32_t lds = std::max(planes_lds_bytes(v, tf.K), order ? kOrderLdsBytes : 0u);
  const unsigned grid = (unsigned)((nb + kPrepThreads - 1) / kPrepThreads) + (order ? 1u : 0u);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_occupancy_planes),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_occupancy_planes, dim3(grid), dim3(kPrepThreads), lds, s, v, tf, bits, o, order);
  return hipGetLastError();
}

hipError_t launch_occupancy_planes(const VolConst &v, const TfConst &tf, uint32_t *bits, hipStream_t s) {
  return launch_planes(v, tf, bits, OrderArgs{}, nullptr, s);
}

hipError_t launch_planes_and_order(const RenderArgs &a, uint32_t *bits, int32_t *order, hipStream_t s) {
  return launch_planes(a.vol, a.tf, bits, order_args(a), order, s);
}

}  // namespace vr
