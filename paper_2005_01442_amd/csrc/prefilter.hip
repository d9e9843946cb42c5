// prefilter.hip -- interpolating cubic B-spline coefficients (gfx950).
//
// Along every axis line the coefficients solve
//   (c[i-1] + 4 c[i] + c[i+1]) / 6 = v[i],  c[-1] = c[0], c[n] = c[n-1]
// (diagonal 5 in the end rows).  The elimination's pivots depend on the index
// alone: with u[i] = 1 / pivot[i] (u[0] = 1/5, u[i] = 1 / (4 - u[i-1]), the
// last row 1 / (5 - u[n-2])) a line is
//   forward   y[i] = (6 v[i] - y[i-1]) u[i]
//   backward  c[i] = y[i] - u[i] c[i+1]   (c[n-1] = y[n-1]),
// two first-order linear recurrences.  u[i] settles to 2 - sqrt(3) within
// fp32 by i = 8; PrefilterCoef carries the first kPivots in kernel arguments.
//
// What bounds it: memory (the volume is read once and the fp32 output written
// three times and read twice; a thread that sweeps a whole line waits for
// memory twice per voxel and, along x, reads with a row's stride between
// lanes).  So a line is cut into segments, one per thread: each solves its
// recurrence in registers with a zero carry-in, the segments' ends are combined
// (a recurrence over a segment is the affine map carry -> end + P carry, P the
// product of its factors), and the segment is swept again from its carry: the
// second sweep rounds as a sweep of the whole line does (adding the carry's
// share to the first sweep's values instead doubled the error).  Every voxel
// is read and written once per axis, in coalesced rows, with up to 64 loads in
// flight per thread.  512x512x400 int16: 4.55 ms with one thread per line,
// 0.52 ms now (x 0.145 ms, y and z 0.19-0.2 ms each: 4.2-4.4 TB/s, a large
// copy reaches 4.7).  Running x and y slab by slab, for the y pass to find its
// slab in the caches, measured slower (0.68 ms with 64 MiB slabs).
#include <algorithm>

#include "vr_internal.h"

namespace vr {

constexpr int kPivots = 16;
struct PrefilterCoef {
  float u[kPivots];
};

// 1 / pivot of row i with diagonal `diag` there (4, or 5 in the last row), FP64.
static double pivot(int i, double diag) {
  double u = 0.2;
  if (i == 0) return u;
  for (int k = 1; k < i && k < 64; ++k) u = 1.0 / (4.0 - u);  // (settled long before 64)
  return 1.0 / (diag - u);
}
static float last_pivot(int n) { return (float)pivot(n - 1, 5.0); }

constexpr int kRowMax = 16 * kWaveSize;        // x: voxels of a row (at most 16 per lane of its wavefront)
constexpr int kSeg = 64;                       // y, z: voxels of a line per thread
constexpr int kLineWaves = 16;                 // y, z: wavefronts (segments of a line) per workgroup
constexpr int kLineMax = kSeg * kLineWaves;
constexpr int kLoadBatch = 8;

// u of voxel j of the segment that starts at i0 (a constant array index: the
// factors stay in scalar registers); row i of a line of n voxels is the last.
__device__ inline float segment_pivot(const PrefilterCoef &c, int i0, int j) {
  return i0 == 0 && j < kPivots ? c.u[j] : c.u[kPivots - 1];
}

template <int DT>
__device__ inline float voxel_f32(const void *src, int64_t i) {
  if constexpr (DT == kF32) return reinterpret_cast<const float *>(src)[i];
  if constexpr (DT == kI16) return (float)reinterpret_cast<const int16_t *>(src)[i];
  return (float)reinterpret_cast<const uint16_t *>(src)[i];
}

// EM consecutive voxels from element i as fp32: loads of up to 16 bytes,
// aligned to a voxel only (the memcpy's compile to global_load_dwordx4).
template <int DT, int EM>
__device__ inline void load_run(const void *src, int64_t i, float v[EM]) {
  if constexpr (EM == 1) {
    v[0] = voxel_f32<DT>(src, i);
  } else if constexpr (DT == kF32) {
    __builtin_memcpy(v, reinterpret_cast<const float *>(src) + i, EM * 4);
  } else {
    uint32_t w[EM / 2];
    __builtin_memcpy(w, reinterpret_cast<const uint16_t *>(src) + i, EM * 2);
#pragma unroll
    for (int j = 0; j < EM / 2; ++j) {
      v[2 * j] = DT == kI16 ? (float)(int16_t)(w[j] & 0xffffu) : (float)(w[j] & 0xffffu);
      v[2 * j + 1] = DT == kI16 ? (float)((int32_t)w[j] >> 16) : (float)(w[j] >> 16);
    }
  }
}

// Product of two runs' factors, kept from underflowing to 0: the carry of a
// line that holds an infinity stays an infinity.
constexpr float kLeastFactor = 1.17549435e-38f;
__device__ inline float carry_product(float p, float q) {
  const float r = p * q;
  return p == 0.0f || q == 0.0f ? 0.0f : copysignf(fmaxf(fabsf(r), kLeastFactor), r);
}
// `end` plus what a run of factor p passes on of `carry`.  A factor at the floor
// stands for one that has underflowed: it passes on nothing finite, so that the
// coefficients far from any voxel other than zero are zero (as sweeps of the
// whole line give, and as the blocks there have to be to count as empty).
__device__ inline float pass_on(float p, float carry, float end) {
  const bool none = fabsf(p) <= kLeastFactor && __builtin_isfinite(carry);
  return none ? end : fmaf(p, carry, end);
}

// x axis, with the conversion to fp32: W lanes per row, lane l of them solves
// voxels [l EM, l EM + EM), read and written as wide runs, and the carries
// come from scans of the lanes' affine maps.  (Staging the row through LDS
// for single-voxel coalesced accesses, any number of voxels per lane:
// 255 us
// against 145 us on 512x512x400 int16.)  W is the whole wavefront from rows of
// 33 voxels on, else the power of two that holds the row: a launch has fewer
// than 2 threads per voxel, below the 2^32 a grid may have, and few lanes idle.
template <int DT, int EM, int W>
__global__ __launch_bounds__(kWgSize) void k_prefilter_rows(const void *src, float *dst, int nx, int64_t rows,
                                                            const PrefilterCoef coef, float last) {
  constexpr int kHead = kPivots / EM;  // lanes whose pivots are not settled
  __shared__ float pivots[kPivots + EM];
  if (threadIdx.x < kPivots + EM) pivots[threadIdx.x] = coef.u[min((int)threadIdx.x, kPivots - 1)];
  __syncthreads();
  const int lane = threadIdx.x % W;
  const int64_t row = (int64_t)blockIdx.x * (kWgSize / W) + threadIdx.x / W;
  if (row >= rows) return;  // uniform over the row's lanes; no barrier follows
  const int i0 = lane * EM, cnt = nx - i0;  // this lane's voxels in the row: min(cnt, EM)
  const int64_t base = row * nx + i0;
  // voxels past the row's end have factor 0: they carry nothing either way
  float v[EM], u[EM];
#pragma unroll
  for (int j = 0; j < EM; ++j) {
    v[j] = 0.0f;
    u[j] = pivots[min(lane, kHead) * EM + j];
  }
  if (cnt >= EM) {
    load_run<DT, EM>(src, base, v);
  } else {
#pragma unroll
    for (int j = 0; j < EM; ++j)
      if (j < cnt) v[j] = voxel_f32<DT>(src, base + j);
  }
  if (cnt <= EM) {  // the row's last voxel is here or before
#pragma unroll
    for (int j = 0; j < EM; ++j) u[j] = j == cnt - 1 ? last : (j < cnt ? u[j] : 0.0f);
  }
  float y = 0.0f, P = 1.0f;
#pragma unroll
  for (int j = 0; j < EM; ++j) {
    v[j] *= 6.0f;
    y = (v[j] - y) * u[j];
    P *= -u[j];
  }
#pragma unroll
  for (int off = 1; off < W; off <<= 1) {
    const float a = __shfl_up(P, off, W), b = __shfl_up(y, off, W);
    if (lane >= off) {
      y = pass_on(P, b, y);
      P = carry_product(P, a);
    }
  }
  y = __shfl_up(y, 1, W);
  if (lane == 0) y = 0.0f;
#pragma unroll
  for (int j = 0; j < EM; ++j) {
    y = (v[j] - y) * u[j];
    v[j] = y;
  }
  if (cnt <= EM) {  // the last row takes nothing from beyond
#pragma unroll
    for (int j = 0; j < EM; ++j) {
      u[j] = j < cnt - 1 ? u[j] : 0.0f;
      v[j] = j < cnt ? v[j] : 0.0f;
    }
  }
  float x = 0.0f, Q = 1.0f;
#pragma unroll
  for (int j = EM - 1; j >= 0; --j) {
    x = v[j] - u[j] * x;
    Q *= -u[j];
  }
#pragma unroll
  for (int off = 1; off < W; off <<= 1) {
    const float a = __shfl_down(Q, off, W), b = __shfl_down(x, off, W);
    if (lane + off < W) {
      x = pass_on(Q, b, x);
      Q = carry_product(Q, a);
    }
  }
  x = __shfl_down(x, 1, W);
  if (lane == W - 1) x = 0.0f;
#pragma unroll
  for (int j = EM - 1; j >= 0; --j) {
    x = v[j] - u[j] * x;
    v[j] = x;
  }
  if (cnt >= EM) {
    __builtin_memcpy(dst + base, v, EM * 4);
  } else {
#pragma unroll
    for (int j = 0; j < EM; ++j)
      if (j < cnt) dst[base + j] = v[j];
  }
}

// y and z axes, in place: a workgroup owns 64 neighbouring lines (lanes along
// x, so every access is a coalesced row), wavefront w their segment
// [w len, w len + len).  All of a line's reads happen before the barrier that
// precedes its first write, and lines are independent.
__global__ __launch_bounds__(kLineWaves *kWaveSize) void k_prefilter_lines(float *vol, int nx, int64_t lines, int n,
                                                                          int64_t stride, int64_t plane, int len,
                                                                          const PrefilterCoef coef, float last) {
  __shared__ float ends[kLineWaves][kWaveSize];  // a segment's last y, then its first c
  __shared__ float prod[kLineWaves];             // the product of its factors
  const int lane = threadIdx.x % kWaveSize;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWaveSize));
  const int waves = (int)(blockDim.x / kWaveSize);
  const int64_t line = (int64_t)blockIdx.x * kWaveSize + lane;
  const bool on = line < lines;
  const int64_t first = min(line, lines - 1);  // lanes past the last line repeat it and store nothing
  float *p = vol + (first / nx) * plane + first % nx;
  const int i0 = wave * len, cnt = min(len, n - i0);  // uniform, cnt >= 1
  float v[kSeg];
#pragma unroll
  for (int j0 = 0; j0 < kSeg; j0 += kLoadBatch)
    if (j0 < cnt) {
#pragma unroll
      for (int j = j0; j < j0 + kLoadBatch; ++j) v[j] = p[(int64_t)(i0 + min(j, cnt - 1)) * stride];
    }
  float y = 0.0f;
  if (waves > 1) {  // the carry into this segment
    float P = 1.0f;
#pragma unroll
    for (int j = 0; j < kSeg; ++j)
      if (j < cnt) {
        const float u = i0 + j == n - 1 ? last : segment_pivot(coef, i0, j);
        y = (6.0f * v[j] - y) * u;
        P *= -u;
      }
    ends[wave][lane] = y;
    if (lane == 0) prod[wave] = P;
    __syncthreads();
    y = 0.0f;
    for (int q = 0; q < wave; ++q) y = fmaf(prod[q], y, ends[q][lane]);
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kSeg; ++j)
    if (j < cnt) {
      const float u = i0 + j == n - 1 ? last : segment_pivot(coef, i0, j);
      y = (6.0f * v[j] - y) * u;
      v[j] = y;
    }
  float x = 0.0f;
  if (waves > 1) {
    float Q = 1.0f;
#pragma unroll
    for (int j = kSeg - 1; j >= 0; --j)
      if (j < cnt) {
        const float u = i0 + j == n - 1 ? 0.0f : segment_pivot(coef, i0, j);
        x = v[j] - u * x;
        Q *= -u;
      }
    ends[wave][lane] = x;
    if (lane == 0) prod[wave] = Q;
    __syncthreads();
    x = 0.0f;
    for (int q = waves - 1; q > wave; --q) x = fmaf(prod[q], x, ends[q][lane]);
  }
#pragma unroll
  for (int j = kSeg - 1; j >= 0; --j)
    if (j < cnt) {
      const float u = i0 + j == n - 1 ? 0.0f : segment_pivot(coef, i0, j);
      x = v[j] - u * x;
      if (on) p[(int64_t)(i0 + j) * stride] = x;
    }
}

// Lines longer than kLineMax: one thread sweeps a line, in place.
__global__ __launch_bounds__(kWgSize) void k_prefilter_serial(float *vol, int nx, int64_t lines, int n, int64_t stride,
                                                              int64_t plane, const PrefilterCoef coef, float last) {
  const int64_t line = (int64_t)blockIdx.x * kWgSize + threadIdx.x;
  if (line >= lines) return;
  float *p = vol + (line / nx) * plane + line % nx;
  float y = 0.0f;
  for (int i = 0; i < n; ++i) {
    y = (6.0f * p[(int64_t)i * stride] - y) * (i == n - 1 ? last : coef.u[min(i, kPivots - 1)]);
    p[(int64_t)i * stride] = y;
  }
  for (int i = n - 2; i >= 0; --i) {
    y = p[(int64_t)i * stride] - coef.u[min(i, kPivots - 1)] * y;
    p[(int64_t)i * stride] = y;
  }
}

// Copy a volume of any dtype into fp32.
template <int DT>
__global__ __launch_bounds__(kWgSize) void k_to_f32(const void *src, float *dst, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kWgSize + threadIdx.x; i < n; i += (int64_t)gridDim.x * kWgSize)
    dst[i] = voxel_f32<DT>(src, i);
}

template <int DT, int EM, int W>
static void launch_rows_as(const VolConst &v, float *out, const PrefilterCoef &coef, hipStream_t s) {
  const int64_t rows = (int64_t)v.ny * v.nz, per_wg = kWgSize / W;
  hipLaunchKernelGGL((k_prefilter_rows<DT, EM, W>), dim3((unsigned)((rows + per_wg - 1) / per_wg)), dim3(kWgSize), 0, s,
                     v.data, out, v.nx, rows, coef, last_pivot(v.nx));
}

template <int DT>
static void launch_rows(const VolConst &v, float *out, const PrefilterCoef &coef, hipStream_t s) {
  const int nx = v.nx;
  const int64_t rows = (int64_t)v.ny * v.nz;
  if (nx == 1 || nx > kRowMax) {  // (a line of one voxel is its own solution)
    const int64_t n = rows * nx, g = std::min<int64_t>((n + kWgSize - 1) / kWgSize, 65536);
    hipLaunchKernelGGL(k_to_f32<DT>, dim3((unsigned)g), dim3(kWgSize), 0, s, v.data, out, n);
    if (nx > 1)
      hipLaunchKernelGGL(k_prefilter_serial, dim3((unsigned)((rows + kWgSize - 1) / kWgSize)), dim3(kWgSize), 0, s, out,
                         1, rows, nx, (int64_t)1, (int64_t)nx, coef, last_pivot(nx));
    return;
  }
  // the fewest voxels per lane (1, 4, 8 or 16) and lanes that hold the row (with
  // a whole wavefront per row, all three axes of 20x1024x1024 int16 took 395 us,
  // 245 now; of 2x4096x4096 8.4 ms, 4.0 now)
  if (nx <= 2) return launch_rows_as<DT, 1, 2>(v, out, coef, s);
  if (nx <= 4) return launch_rows_as<DT, 1, 4>(v, out, coef, s);
  if (nx <= 8) return launch_rows_as<DT, 1, 8>(v, out, coef, s);
  if (nx <= 16) return launch_rows_as<DT, 1, 16>(v, out, coef, s);
  if (nx <= 32) return launch_rows_as<DT, 1, 32>(v, out, coef, s);
  if (nx <= kWaveSize) return launch_rows_as<DT, 1, kWaveSize>(v, out, coef, s);
  if (nx <= 4 * kWaveSize) return launch_rows_as<DT, 4, kWaveSize>(v, out, coef, s);
  if (nx <= 8 * kWaveSize) return launch_rows_as<DT, 8, kWaveSize>(v, out, coef, s);
  return launch_rows_as<DT, 16, kWaveSize>(v, out, coef, s);
}

// `lines` lines of n voxels `stride` apart; line l starts at (l / nx) plane + l % nx.
static void launch_lines(float *out, int nx, int64_t lines, int n, int64_t stride, int64_t plane,
                         const PrefilterCoef &coef, hipStream_t s) {
  if (n == 1) return;
  if (n > kLineMax) {
    hipLaunchKernelGGL(k_prefilter_serial, dim3((unsigned)((lines + kWgSize - 1) / kWgSize)), dim3(kWgSize), 0, s, out,
                       nx, lines, n, stride, plane, coef, last_pivot(n));
    return;
  }
  const int segs = (n + kSeg - 1) / kSeg, len = (n + segs - 1) / segs, waves = (n + len - 1) / len;
  hipLaunchKernelGGL(k_prefilter_lines, dim3((unsigned)((lines + kWaveSize - 1) / kWaveSize)), dim3(waves * kWaveSize),
                     0, s, out, nx, lines, n, stride, plane, len, coef, last_pivot(n));
}

hipError_t launch_prefilter(const VolConst &v, float *out, hipStream_t s) {
  PrefilterCoef coef;
  for (int i = 0; i < kPivots; ++i) coef.u[i] = (float)pivot(i, 4.0);
  switch (v.dtype) {
  case kU16: launch_rows<kU16>(v, out, coef, s); break;
  case kI16: launch_rows<kI16>(v, out, coef, s); break;
  default: launch_rows<kF32>(v, out, coef, s); break;
  }
  // (the passes along y and z read what this one writes)
  if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  const int64_t nx = v.nx, nxy = nx * v.ny;
  launch_lines(out, v.nx, nx * v.nz, v.ny, nx, nxy, coef, s);
  launch_lines(out, v.nx, nxy, v.nz, nxy, nx, coef, s);
  return hipGetLastError();
}

}  // namespace vr
