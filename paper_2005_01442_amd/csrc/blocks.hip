// blocks.hip -- block min/max build and TF-dependent block occupancy (gfx950).
//
// The paper decomposes the volume into fixed-size blocks (smaller at the far
// faces) that overlap by the voxels a cubic stencil reads, and drops blocks
// with nothing visible (Section 2, block decomposition, Fig. 3, "Pros" (a),
// (b)).  Here a block is the cell range [bE, bE+E) per axis; its footprint
// [bE-1, bE+E+1] (clamped) is every voxel a tricubic sample with its cell in
// the block can read, and the per-block (min, max) over that footprint,
// together with the TF, decides whether the block can hold a visible sample.
#include "vr_internal.h"

namespace vr {

// A block's range and, beside it, the range widened for Catmull-Rom samples,
// [lo - w (hi - lo), hi + w (hi - lo)] (fused, fp32).
__device__ inline void store_range(float2 *out, float2 *wide, int64_t b, float lo, float hi, float w) {
  const float d = hi - lo;
  out[b] = make_float2(lo, hi);
  wide[b] = make_float2(fmaf(-w, d, lo), fmaf(w, d, hi));
}

// A workgroup of eight wavefronts per row of blocks in x: the x-rows of the
// footprint ([bE - 1, bE + E + 1] in y and z, clamped) are streamed in z order,
// the wavefronts taking every eighth row, four rows per trip (their loads in
// flight together).  A lane holds eight
// consecutive voxels (kRun) of a row, E / 8 lanes a block; the footprint's
// apron along x (one voxel before the block, two after it) comes from the
// neighbouring lanes.  The wavefronts are combined in LDS at the end of a pass
// over 512 voxels of x.
//
// What bounds it: the volume read once, so every voxel is loaded in 16-byte
// runs that need only a voxel's alignment: rows of any length and parity take
// the same path (one lane per 8 voxels with single-voxel loads, whose lanes
// lie 16 bytes apart, took 218 us on 511x509x397 int16 where this takes 51 us: 4.1 of the 4.7 TB/s
// a large copy reaches).
// Neighbouring blocks in z share three planes, which the caches hold: four
// blocks in z per workgroup, each plane read once, took 858 us on 1024^3 int16,
// two 701, one 624 (fewer workgroups and selects per row).
// The run of a row's last lane starts at the row's eighth voxel from its end and
// is shifted into place by the same (uniform) count in every row.
constexpr int kRun = 8;
constexpr int kMinmaxRows = 4;   // rows per wavefront trip (2 to 8 measured; 8 slower)
constexpr int kMinmaxThreads = 512;  // eight wavefronts: more rows in flight per row of blocks

// Lane i takes lane i - 1's (left) or i + 1's (right) value; the end lane keeps `own`.
__device__ inline uint32_t from_left(uint32_t x, uint32_t own) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)own, (int)x, 0x138, 0xF, 0xF, false);  // wave_shr:1
}
__device__ inline uint32_t from_right(uint32_t x, uint32_t own) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)own, (int)x, 0x130, 0xF, 0xF, false);  // wave_shl:1
}

// Eight voxels of a row and a running (min, max).  16-bit voxels stay packed
// integers, two per register (v_pk_min / v_pk_max), exact, and become floats
// once per pass; fp32 voxels are floats throughout.
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

template <typename T, typename V, int LO, int HI>
struct Run16 {
  static constexpr int kWords = 4;  // registers of a run
  struct Range {
    V mn = {(T)HI, (T)HI}, mx = {(T)LO, (T)LO};
    __device__ inline void add(uint32_t w) {
      mn = __builtin_elementwise_min(mn, __builtin_bit_cast(V, w));
      mx = __builtin_elementwise_max(mx, __builtin_bit_cast(V, w));
    }
    __device__ inline void add(const Range &r) {
      mn = __builtin_elementwise_min(mn, r.mn);
      mx = __builtin_elementwise_max(mx, r.mx);
    }
    __device__ inline float lo() const { return (float)min(mn.x, mn.y); }
    __device__ inline float hi() const { return (float)max(mx.x, mx.y); }
  };
  // a voxel as one or both halves of a register
  __device__ static inline uint32_t voxel(const T *p) { return (uint32_t)(uint16_t)*p * 0x10001u; }
  __device__ static inline uint32_t last(const uint32_t w[4]) { return __builtin_amdgcn_perm(w[3], w[3], 0x03020302u); }
  // the run moved down by s voxels (uniform), `end` moving in
  __device__ static inline void shift(uint32_t w[4], int s, uint32_t end) {
    if (s & 1) {
      w[0] = __builtin_amdgcn_alignbit(w[1], w[0], 16);
      w[1] = __builtin_amdgcn_alignbit(w[2], w[1], 16);
      w[2] = __builtin_amdgcn_alignbit(w[3], w[2], 16);
      w[3] = end;  // (its low half held the last voxel)
    }
    if (s & 2) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = end; }
    if (s & 4) { w[0] = w[2]; w[1] = w[3]; w[2] = w[3] = end; }
  }
  // the apron: the voxel before the run (the left lane's last) and the two
  // after it (the right lane's first two, one register)
  __device__ static inline uint32_t before(const uint32_t w[4]) { return from_left(last(w), (w[0] & 0xffffu) | (w[0] << 16)); }
  __device__ static inline void after(const uint32_t w[4], uint32_t &a, uint32_t &b) { a = b = from_right(w[0], last(w)); }
};

template <typename T> struct Run;
template <> struct Run<int16_t> : Run16<short, s16x2, -32768, 32767> {};
template <> struct Run<uint16_t> : Run16<unsigned short, u16x2, 0, 65535> {};
template <> struct Run<float> {
  static constexpr int kWords = 8;
  struct Range {
    float mn = INFINITY, mx = -INFINITY;
    __device__ inline void add(uint32_t w) {
      mn = fminf(mn, __builtin_bit_cast(float, w));
      mx = fmaxf(mx, __builtin_bit_cast(float, w));
    }
    __device__ inline void add(const Range &r) {
      mn = fminf(mn, r.mn);
      mx = fmaxf(mx, r.mx);
    }
    __device__ inline float lo() const { return mn; }
    __device__ inline float hi() const { return mx; }
  };
  __device__ static inline uint32_t voxel(const float *p) { return __builtin_bit_cast(uint32_t, *p); }
  __device__ static inline uint32_t last(const uint32_t w[8]) { return w[7]; }
  __device__ static inline void shift(uint32_t w[8], int s, uint32_t end) {
#pragma unroll
    for (int b = 1; b < 8; b *= 2)
      if (s & b) {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = i + b < 8 ? w[i + b < 8 ? i + b : 0] : end;
      }
  }
  __device__ static inline uint32_t before(const uint32_t w[8]) { return from_left(w[7], w[0]); }
  __device__ static inline void after(const uint32_t w[8], uint32_t &a, uint32_t &b) {
    a = from_right(w[0], w[7]);
    b = from_right(w[1], w[7]);
  }
};

// Block edges of 8 and more, rows of at least kRun voxels.
template <typename T>
__global__ __launch_bounds__(kMinmaxThreads) void k_block_minmax(const VolConst v, float2 *out, float2 *wide, float widen) {
  typedef Run<T> R;
  constexpr int kWaves = kMinmaxThreads / kWaveSize;
  __shared__ float smin[kWaves][kWaveSize], smax[kWaves][kWaveSize];
  // XCD-aware: workgroup i runs on XCD i mod 8; each XCD takes a contiguous
  // run of items, neighbouring rows of blocks in y side by side
  const int nitems = v.nby * v.nbz, per_xcd = (nitems + kXcds - 1) / kXcds;
  const int q = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
  if (q >= nitems) return;
  const int E = v.edge, lpb_shift = v.edge_shift - 3, lpb = 1 << lpb_shift;  // lanes per block
  const int by = q % v.nby, bz = q / v.nby;
  const int y0 = max(by * E - 1, 0), y1 = min(by * E + E + 1, v.ny - 1);
  const int z0 = max(bz * E - 1, 0), z1 = min(bz * E + E + 1, v.nz - 1);
  const int ny = y1 - y0 + 1, rows = ny * (z1 - z0 + 1);
  // the wavefront index, as a uniform value: the row walk below stays scalar
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWaveSize));
  const int lane = threadIdx.x % kWaveSize;
  const T *base = reinterpret_cast<const T *>(v.data);
  const int per_pass = kWaveSize >> lpb_shift;  // blocks per pass
  const bool first = (lane & (lpb - 1)) == 0, final = (lane & (lpb - 1)) == lpb - 1;  // of its block
  const int ragged = v.nx % kRun;
  for (int bx0 = 0; bx0 < v.nbx; bx0 += per_pass) {
    const int xa = bx0 * E + lane * kRun;  // this lane's first voxel
    const int xs = min(xa, v.nx - kRun);   // the run it loads
    const bool more = bx0 * E + kWaveSize * kRun < v.nx;  // uniform: voxels past the pass
    typename R::Range range;
    // footprint row r = (y - y0) + ny (z - z0), walked by increments (no
    // division per row); rows past the last repeat it, which changes nothing
    int r = wave, y = y0 + wave % ny, z = z0 + wave / ny;
    while (r < rows) {
#pragma unroll
      for (int u = 0; u < kMinmaxRows; ++u) {
        const bool in = r < rows;
        const int yy = in ? y : y1, zz = in ? z : z1;
        const T *row = base + ((size_t)zz * (size_t)v.ny + (size_t)yy) * (size_t)v.nx;
        uint32_t w[R::kWords];
        __builtin_memcpy(w, row + xs, kRun * sizeof(T));
        if (ragged != 0 && !more) {  // uniform: the row ends in this pass
          uint32_t t[R::kWords];
          const uint32_t end = R::last(w);
#pragma unroll
          for (int i = 0; i < R::kWords; ++i) t[i] = w[i];
          R::shift(t, kRun - ragged, end);
#pragma unroll
          for (int i = 0; i < R::kWords; ++i) w[i] = xa == xs ? w[i] : (xa < v.nx ? t[i] : end);
        }
        uint32_t lo = R::before(w), hi0, hi1;
        R::after(w, hi0, hi1);
        if (bx0 > 0 && lane == 0) lo = R::voxel(row + xa - 1);
        if (more && lane == kWaveSize - 1) {
          const uint32_t p = R::voxel(row + min(xa + kRun, v.nx - 1)), n = R::voxel(row + min(xa + kRun + 1, v.nx - 1));
          hi0 = p;
          hi1 = n;
        }
#pragma unroll
        for (int i = 0; i < R::kWords; ++i) range.add(w[i]);
        range.add(first ? lo : w[0]);
        range.add(final ? hi0 : w[0]);
        range.add(final ? hi1 : w[0]);
        r += kWaves;
        y += kWaves;
        while (y > y1) {
          y -= ny;
          ++z;
        }
      }
    }
    float fmn = range.lo(), fmx = range.hi();
    for (int off = 1; off < lpb; off <<= 1) {
      fmn = fminf(fmn, __shfl_xor(fmn, off, kWaveSize));
      fmx = fmaxf(fmx, __shfl_xor(fmx, off, kWaveSize));
    }
    if (first) {
      smin[wave][lane >> lpb_shift] = fmn;
      smax[wave][lane >> lpb_shift] = fmx;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < per_pass; i += kMinmaxThreads) {
      const int b = bx0 + i;
      float m0 = smin[0][i], m1 = smax[0][i];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        m0 = fminf(m0, smin[w][i]);
        m1 = fmaxf(m1, smax[w][i]);
      }
      if (b < v.nbx) store_range(out, wide, ((int64_t)bz * v.nby + by) * v.nbx + b, m0, m1, widen);
    }
    __syncthreads();
  }
}

// Any edge and row length (edges of 4, rows of fewer than kRun voxels): eight
// lanes per block, each every eighth plane of its footprint (with one lane per
// block a 97x81x73 volume waited for 343 loads in a row: 33 us, 13 us now).
template <typename T>
__global__ __launch_bounds__(kWgSize) void k_block_minmax_small(const VolConst v, float2 *out, float2 *wide, float widen) {
  const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  const int64_t at = ((int64_t)blockIdx.x * kWgSize + threadIdx.x) / 8, b = min(at, nb - 1);
  const int E = v.edge, n[3] = {v.nx, v.ny, v.nz};
  const int bc[3] = {(int)(b % v.nbx), (int)(b / v.nbx % v.nby), (int)(b / ((int64_t)v.nbx * v.nby))};
  int lo[3], hi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = max(bc[a] * E - 1, 0);
    hi[a] = min(bc[a] * E + E + 1, n[a] - 1);
  }
  const T *base = reinterpret_cast<const T *>(v.data);
  float mn = INFINITY, mx = -INFINITY;
  for (int z = lo[2] + (int)(threadIdx.x % 8); z <= hi[2]; z += 8)
    for (int y = lo[1]; y <= hi[1]; ++y) {
      const T *row = base + ((size_t)z * (size_t)v.ny + (size_t)y) * (size_t)v.nx;
      for (int x = lo[0]; x <= hi[0]; ++x) {
        const float f = (float)row[x];
        mn = fminf(mn, f);
        mx = fmaxf(mx, f);
      }
    }
#pragma unroll
  for (int off = 1; off < 8; off <<= 1) {
    mn = fminf(mn, __shfl_xor(mn, off, kWaveSize));
    mx = fmaxf(mx, __shfl_xor(mx, off, kWaveSize));
  }
  if (at < nb && threadIdx.x % 8 == 0) store_range(out, wide, b, mn, mx, widen);
}

template <typename T>
static void launch_minmax(const VolConst &v, float2 *out, float2 *wide, float widen, hipStream_t s) {
  if (v.edge < kRun || v.nx < kRun) {
    const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
    hipLaunchKernelGGL(k_block_minmax_small<T>, dim3((unsigned)((8 * nb + kWgSize - 1) / kWgSize)), dim3(kWgSize), 0, s,
                       v, out, wide, widen);
    return;
  }
  const unsigned grid = (unsigned)(((int64_t)v.nby * v.nbz + kXcds - 1) / kXcds * kXcds);
  hipLaunchKernelGGL(k_block_minmax<T>, dim3(grid), dim3(kMinmaxThreads), 0, s, v, out, wide, widen);
}

hipError_t launch_block_minmax(const VolConst &v, float2 *out, float2 *wide, float widen, hipStream_t s) {
  switch (v.dtype) {
  case kU16: launch_minmax<uint16_t>(v, out, wide, widen, s); break;
  case kI16: launch_minmax<int16_t>(v, out, wide, widen, s); break;
  case kF32: launch_minmax<float>(v, out, wide, widen, s); break;
  default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// One thread per block; the TF and its prefix counts sit in LDS.  The same
// decision (range_occupied) is taken on the fly by the render kernels.
__global__ __launch_bounds__(kWgSize) void k_block_occupancy(const VolConst v, const TfConst tf, uint8_t *occ) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  TfShared s = carve_tf(lds, tf.K);
  load_tf(s, tf);
  const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  const int64_t b = (int64_t)blockIdx.x * kWgSize + threadIdx.x;
  if (b < nb) occ[b] = block_occupied(v, s, tf, (int)b) ? 1 : 0;
}

hipError_t launch_block_occupancy(const VolConst &v, const TfConst &tf, uint8_t *occ, hipStream_t s) {
  int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  unsigned grid = (unsigned)((nb + kWgSize - 1) / kWgSize);
  hipLaunchKernelGGL(k_block_occupancy, dim3(grid), dim3(kWgSize), tf_lds_bytes(tf.K), s, v, tf, occ);
  return hipGetLastError();
}

// One thread per block, one ballot per 64 blocks; bits past the last block
// are zero.
__global__ __launch_bounds__(kWgSize) void k_occupancy_bits(const VolConst v, const TfConst tf, uint32_t *bits) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  TfShared s = carve_tf(lds, tf.K);
  load_tf(s, tf);
  const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  const int64_t b = (int64_t)blockIdx.x * kWgSize + threadIdx.x;
  const unsigned long long m = __ballot(b < nb && block_occupied(v, s, tf, (int)b));
  const int lane = threadIdx.x % kWaveSize;
  if ((lane == 0 || lane == 32) && b < nb) bits[b >> 5] = lane == 0 ? (uint32_t)m : (uint32_t)(m >> 32);
}

hipError_t launch_occupancy_bits(const VolConst &v, const TfConst &tf, uint32_t *bits, hipStream_t s) {
  VolConst vm = v;
  vm.occ = nullptr;  // decide from minmax
  const int64_t nb = (int64_t)v.nbx * v.nby * v.nbz;
  const unsigned grid = (unsigned)((nb + kWgSize - 1) / kWgSize);
  hipLaunchKernelGGL(k_occupancy_bits, dim3(grid), dim3(kWgSize), tf_lds_bytes(tf.K), s, vm, tf, bits);
  return hipGetLastError();
}

__global__ __launch_bounds__(kWgSize) void k_fill_zero(float *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kWgSize + threadIdx.x; i < n; i += (int64_t)gridDim.x * kWgSize) p[i] = 0.0f;
}

hipError_t launch_fill_zero(float *p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t g = (n + kWgSize - 1) / kWgSize;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)g), dim3(kWgSize), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace vr
