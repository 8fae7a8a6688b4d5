// Reduced-precision staging of the tall data: the BF16 and FP8 E4M3 copies
// that the low-precision forms of the sketch and of the data passes read.
//
//  * BF16: round to nearest even on the 16 discarded bits of the FP32 value;
//    a NaN stays a quiet NaN with its sign and upper payload.
//  * FP8 E4M3 (OCP; bias 7, 3 mantissa bits, no infinities, 448 largest):
//    each column j is scaled by the smallest power of two 2^e_j with
//    max_i |x_ij| <= 448 2^e_j (exact comparisons), then every entry is
//    rounded to the nearest E4M3 value, ties to the even mantissa,
//    saturating at +-448.  Undoing a power-of-two scale is exact, so a
//    sketch of the codes times the column scales equals the sketch of the
//    staged matrix.
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <cmath>

namespace srp {

// Four consecutive elements read or written at once.  The vectors are only
// element-aligned (a caller's matrix may start anywhere): the hardware takes
// a 16-byte access on any 4-byte boundary.  Nontemporal, since the matrix is
// larger than the caches (maxima of 200000 x 1000 125 us, 162 without; the codes
// 179, 199).
template <class T> struct StageVec;
template <> struct StageVec<float> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct StageVec<bf16> {
  typedef unsigned short type __attribute__((ext_vector_type(4), aligned(2)));
};
__device__ __forceinline__ void stage_load4(const float* p, float (&v)[4]) {
  const auto q = __builtin_nontemporal_load(reinterpret_cast<const StageVec<float>::type*>(p));
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = q[u];
}
__device__ __forceinline__ void stage_load4(const bf16* p, float (&v)[4]) {
  const auto q = __builtin_nontemporal_load(reinterpret_cast<const StageVec<bf16>::type*>(p));
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = __uint_as_float((uint32_t)q[u] << 16);
}

// One read and one write of everything, eight elements a thread as two
// 16-byte loads and one 16-byte store (one element a thread: 423 us a
// call at 200000 x 1000, 2.8 TB/s; so: 216 us, 5.6 TB/s).
__global__ void __launch_bounds__(256) k_stage_bf16(const float* __restrict__ X, int64_t count,
                                                    uint16_t* __restrict__ out) {
  typedef unsigned short u16x8 __attribute__((ext_vector_type(8), aligned(2)));
  const int64_t i = 8 * (blockIdx.x * 256ll + threadIdx.x);
  if (i + 8 <= count) {
    float a[4], b[4];
    stage_load4(X + i, a);
    stage_load4(X + i + 4, b);
    u16x8 o;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      o[u] = bf16_rne_bits(a[u]);
      o[u + 4] = bf16_rne_bits(b[u]);
    }
    *reinterpret_cast<u16x8*>(out + i) = o;
  } else {
    for (int64_t j = i; j < count; ++j) out[j] = bf16_rne_bits(X[j]);
  }
}

// The FP8 kernels walk the matrix in groups of M rows (M a multiple of 4):
// a group is M d / 4 runs of four consecutive elements whatever d is, and
// thread t takes run t of every group it visits, so its four columns
// (4 t + u) mod d stay the same and every access is one vector.  M d / 4 is
// at least a workgroup wide.  Rows past the last whole group are left to
// single elements.
struct StageGeom {
  int M;            // rows of a group
  int runs;         // M d / 4
  int64_t groups;   // whole groups
  int per;          // groups per workgroup
  dim3 grid;
};
static StageGeom stage_geom(int64_t n, int d) {
  StageGeom g;
  g.M = 4 * (int)((256 + (int64_t)d - 1) / d);
  g.runs = (int)((int64_t)g.M * d / 4);
  g.groups = n / g.M;
  const unsigned gx = (unsigned)((g.runs + 255) / 256);
  // about four workgroups a CU (more only write more maxima to join), at
  // least eight groups each
  int64_t gy = std::max<int64_t>(1, 4ll * num_cus() / gx);
  gy = std::min(gy, std::max<int64_t>(1, (g.groups + 7) / 8));
  g.per = (int)((g.groups + gy - 1) / gy);
  gy = g.per > 0 ? (g.groups + g.per - 1) / g.per : 1;
  g.grid = dim3(gx, (unsigned)gy);
  return g;
}

// Maxima of |x| over a workgroup's groups, one for every position of a group.
// A whole read of the matrix, so HBM bounds it: each thread keeps eight vector
// loads in flight (one column per thread with one 4-byte load in flight: 831 us
// at 200000 x 1000).  The maxima go to memory as they are (an atomic maximum a
// column from every thread took 45 us of 183; so: 124 us, 6.5 TB/s, and 5 to
// join them; 200000 x 64, where many threads share a column: the call 715 -> 57).
template <class T>
__global__ void __launch_bounds__(256) k_col_amax(const T* __restrict__ X, int d, StageGeom g,
                                                  float* __restrict__ part) {
  constexpr int UN = 8;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < g.runs) {
    const int64_t stride = (int64_t)g.M * d;
    const int64_t g0 = (int64_t)blockIdx.y * g.per, g1 = min<int64_t>(g.groups, g0 + g.per);
    const T* p = X + g0 * stride + 4ll * t;
    float m[4] = {0.f, 0.f, 0.f, 0.f};
    int64_t q = g0;
    for (; q + UN <= g1; q += UN, p += UN * stride) {
      float v[UN][4];
#pragma unroll
      for (int i = 0; i < UN; ++i) stage_load4(p + i * stride, v[i]);
#pragma unroll
      for (int i = 0; i < UN; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) m[u] = fmaxf(m[u], fabsf(v[i][u]));
    }
    for (; q < g1; ++q, p += stride) {
      float v[4];
      stage_load4(p, v);
#pragma unroll
      for (int u = 0; u < 4; ++u) m[u] = fmaxf(m[u], fabsf(v[u]));
    }
    float4* out = reinterpret_cast<float4*>(part) + (int64_t)blockIdx.y * g.runs + t;
    *out = make_float4(m[0], m[1], m[2], m[3]);
  }
}

// The column maxima from `parts` maxima of every position of a group (64
// positions a workgroup, sixteen slices of the parts), and from the rows past
// the last group, an element a thread in the workgroups past the positions.
// Non-negative floats order like their bit patterns, so an integer atomic
// maximum over a group's few rows is exact whatever the order.
template <class T>
__global__ void __launch_bounds__(1024) k_amax_parts(const T* __restrict__ X, int64_t n, int d, StageGeom g,
                                                     const float* __restrict__ part, int parts,
                                                     uint32_t* __restrict__ amax_bits) {
  __shared__ float q[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, count = 4 * g.runs, wide = (count + 63) / 64;
  const int p = blockIdx.x * 64 + lane;
  if ((int)blockIdx.x >= wide) {
    const int64_t e = g.groups * g.M * d + ((int64_t)blockIdx.x - wide) * 1024 + threadIdx.x;
    if (e < n * d) atomicMax(&amax_bits[e % d], __float_as_uint(fmaxf(0.f, fabsf(load_as<float>(X + e)))));
    return;
  }
  float m = 0.f;
  for (int z = w; z < parts; z += 128) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = z + 16 * u < parts && p < count ? part[(int64_t)(z + 16 * u) * count + p] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) m = fmaxf(m, v[u]);
  }
  q[w][lane] = m;
  __syncthreads();
  if (w == 0 && p < count) {
#pragma unroll
    for (int i = 1; i < 16; ++i) m = fmaxf(m, q[i][lane]);
    atomicMax(&amax_bits[p % d], __float_as_uint(m));
  }
}

// The same from matrices wide enough to give every CU 64 columns: a column a
// lane over all the rows there are of it, the parts' M rows (position p of a
// group is column p mod d of its row p / d) and those past the last group.  No
// atomics, and no workgroup for each of a group's 4 d positions (8 x 1000000:
// 178 us a call, so 57; with the rows past the last group left to one
// workgroup 7 x 1000000 took 1378, so 57).  By positions a width of 1000 has
// four times the workgroups.
template <class T>
__global__ void __launch_bounds__(1024) k_amax_cols(const T* __restrict__ X, int64_t n, int d, StageGeom g,
                                                    const float* __restrict__ part, int parts,
                                                    uint32_t* __restrict__ amax_bits) {
  __shared__ float q[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, W = blockDim.x >> 6;
  const int64_t c = blockIdx.x * 64ll + lane, rows = (int64_t)parts * g.M;
  float m = 0.f;
  if (c < d) {
    for (int64_t r = w; r < rows; r += 8 * W) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = r + u * W < rows ? part[(r + u * W) * d + c] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) m = fmaxf(m, v[u]);
    }
    for (int64_t r = g.groups * g.M + w; r < n; r += W) m = fmaxf(m, fabsf(load_as<float>(X + r * d + c)));
  }
  q[w][lane] = m;
  __syncthreads();
  if (w == 0 && c < d) {
    for (int i = 1; i < W; ++i) m = fmaxf(m, q[i][lane]);
    amax_bits[c] = __float_as_uint(m);
  }
}

__global__ void k_fp8_scales(const uint32_t* __restrict__ amax_bits, int d, double* __restrict__ scales,
                             float* __restrict__ inv_scales) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= d) return;
  const double a = (double)__uint_as_float(amax_bits[c]);
  int e = 0;
  if (a > 0.0) {
    // an infinity: the largest exponent there is (448 2^1015 is still finite),
    // not a search for it from the integer that infinity converts to
    e = (int)fmin(ceil(log2(a / 448.0)), 1016.0);
    while (a > 448.0 * ldexp(1.0, e)) ++e;
    while (a <= 448.0 * ldexp(1.0, e - 1)) --e;
  }
  scales[c] = ldexp(1.0, e);
  inv_scales[c] = ldexpf(1.0f, -e);
}

// E4M3 codes of v[0..3] (nearest, ties to even mantissa, saturating at
// +-448; a NaN saturates with its sign, a negative value that rounds to
// zero gives the positive zero) in the bytes of a word: the hardware's OCP
// conversion after the magnitude is clamped.
__device__ __forceinline__ uint32_t fp8_e4m3_encode4(const float (&v)[4]) {
  float c[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) c[u] = copysignf(fminf(fabsf(v[u]), 448.f), v[u]);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], w, true);
  // bytes 0x80 become 0: bit 7 of each byte survives where its low seven
  // bits are not all zero
  const uint32_t x = (uint32_t)w, low = x & 0x7F7F7F7Fu;
  return low | (x & ((low + 0x7F7F7F7Fu) & 0x80808080u));
}

// A read and a write of everything, as the maxima's read above (one column
// per thread, bytes stored singly: 391 us at 200000 x 1000; so:
// 177 us, 5.6 TB/s).  vec_out: the codes start on a 4-byte boundary (every run
// then does) and leave as words.
template <class T>
__global__ void __launch_bounds__(256) k_stage_fp8(const T* __restrict__ X, int64_t n, int d, StageGeom g,
                                                   const float* __restrict__ inv_scales, int vec_out,
                                                   uint8_t* __restrict__ out) {
  constexpr int UN = 4;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < g.runs) {
    const int64_t stride = (int64_t)g.M * d;
    const int64_t g0 = (int64_t)blockIdx.y * g.per, g1 = min<int64_t>(g.groups, g0 + g.per);
    float is[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) is[u] = inv_scales[(4ll * t + u) % d];
    auto put = [&](float (&v)[4], int64_t e) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] *= is[u];
      const uint32_t w = fp8_e4m3_encode4(v);
      if (vec_out) {
        *reinterpret_cast<uint32_t*>(out + e) = w;
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) out[e + u] = (uint8_t)(w >> (8 * u));
      }
    };
    int64_t e = g0 * stride + 4ll * t, q = g0;
    for (; q + UN <= g1; q += UN, e += UN * stride) {
      float v[UN][4];
#pragma unroll
      for (int i = 0; i < UN; ++i) stage_load4(X + e + i * stride, v[i]);
#pragma unroll
      for (int i = 0; i < UN; ++i) put(v[i], e + i * stride);
    }
    for (; q < g1; ++q, e += stride) {
      float v[4];
      stage_load4(X + e, v);
      put(v, e);
    }
  }
  if (blockIdx.y == 0) {
    const int64_t e0 = g.groups * g.M * d, e1 = n * d;
    for (int64_t e = e0 + t; e < e1; e += (int64_t)gridDim.x * 256) {
      const float v[4] = {load_as<float>(X + e) * inv_scales[e % d], 0.f, 0.f, 0.f};
      out[e] = (uint8_t)fp8_e4m3_encode4(v);
    }
  }
}

__global__ void k_scale_cols(float* __restrict__ A, int64_t rows, int d, const double* __restrict__ scales) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d) return;
  const float sc = (float)scales[c];   // a power of two: the product is exact
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) A[r * d + c] *= sc;
}

int stage_bf16_run(const float* X, int64_t n, int d, uint16_t* out, hipStream_t st) {
  const int64_t count = n * (int64_t)d;
  if (count <= 0) return SRP_OK;
  hipLaunchKernelGGL(k_stage_bf16, dim3((unsigned)((count + 2047) / 2048)), dim3(256), 0, st, X, count, out);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

// The maxima of a group's positions, a set from every row of workgroups.
static size_t stage_parts(const StageGeom& g) { return g.groups > 0 ? (size_t)g.grid.y * 4 * g.runs : 0; }

size_t stage_fp8_ws_bytes(int64_t n, int d) {
  return bytes_of<uint32_t>(d) + bytes_of<float>(d) + bytes_of<float>(stage_parts(stage_geom(n, d)));
}

template <class T>
static int stage_fp8_t(const T* X, int64_t n, int d, uint8_t* out, double* scales, Arena& ws, hipStream_t st) {
  uint32_t* amax = ws.take<uint32_t>(d);
  float* inv = ws.take<float>(d);
  const StageGeom g = stage_geom(n, d);
  float* part = ws.take<float>(stage_parts(g));
  if (!amax || !inv || !part) { set_error("stage_fp8: workspace too small"); return SRP_ENOMEM; }
  const int parts = g.groups > 0 ? (int)g.grid.y : 0;
  if (parts > 0) {
    hipLaunchKernelGGL((k_col_amax<T>), g.grid, dim3(256), 0, st, X, d, g, part);
    SRP_LAUNCH_CHECK();
  }
  if (d >= 64 * num_cus()) {
    const int W = std::min(16, std::max(1, parts * g.M / 4));
    hipLaunchKernelGGL((k_amax_cols<T>), dim3((unsigned)(((int64_t)d + 63) / 64)), dim3(64 * W), 0, st, X, n, d, g,
                       part, parts, amax);
  } else {
    SRP_TRY(fill_i32((int*)amax, d, 0, st));
    const int64_t rest = n * d - g.groups * g.M * d;
    hipLaunchKernelGGL((k_amax_parts<T>), dim3((unsigned)((4 * g.runs + 63) / 64 + (rest + 1023) / 1024)), dim3(1024),
                       0, st, X, n, d, g, part, parts, amax);
  }
  SRP_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_fp8_scales, dim3((d + 255) / 256), dim3(256), 0, st, amax, d, scales, inv);
  SRP_LAUNCH_CHECK();
  hipLaunchKernelGGL((k_stage_fp8<T>), g.grid, dim3(256), 0, st, X, n, d, g, inv, (int)(((uintptr_t)out & 3) == 0),
                     out);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

int stage_fp8_run(const void* X, int dtype, int64_t n, int d, uint8_t* out, double* scales, Arena& ws,
                  hipStream_t st) {
  if (dtype == SRP_F32) return stage_fp8_t((const float*)X, n, d, out, scales, ws, st);
  if (dtype == SRP_BF16) return stage_fp8_t((const bf16*)X, n, d, out, scales, ws, st);
  set_error("stage_fp8: data must be F32 or BF16");
  return SRP_EINVAL;
}

int scale_cols_run(float* A, int64_t rows, int d, const double* scales, hipStream_t st) {
  if (rows <= 0 || d <= 0) return SRP_OK;
  const unsigned gy = (unsigned)std::min<int64_t>(rows, 1024);
  hipLaunchKernelGGL(k_scale_cols, dim3((d + 255) / 256, gy), dim3(256), 0, st, A, rows, d, scales);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

}  // namespace srp
