// Sparse (CSR) data: the O(nnz) CountSketch of Section 3 and the
// per-iteration products of Algorithms CCAopt / LDAopt as sparse-times-
// skinny products, whose cost the paper states in terms of nnz(X) and
// nnz(Y) (Section 3, Table costs; Section 4.5 and 5.5 cost remarks).
//
// Input: row-major CSR (row pointers int64, column indices int32 strictly
// increasing within a row, values F32 or F64).  The products A W read the
// rows.  The products A^T P sort blocks of rows by column in LDS
// (k_csr_tsum), or read the columns of a CSC copy, built once per solve by
// a stable counting sort (column histograms per chunk of rows, a scan per
// column over the chunks, placement row by row inside a chunk), so every
// column lists its rows in ascending order.  Every output is a sum in a
// fixed order (the kernels are bitwise reproducible).  All arithmetic is FP64.
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace srp {

constexpr int kCscChunkMax = 4096;   // largest chunk of rows in the CSC build
// Entries per segment of a column in the products A^T P.
constexpr int kCscSeg = 256;

// ------------------------------------------------------- validation
// Every row: 0 <= ptr[i] <= ptr[i+1] <= nnz, ptr[0] = 0, ptr[n] = nnz,
// columns in [0, d) and strictly increasing.  Entries are only read inside
// [0, nnz), whatever the pointers hold.  Sixteen lanes take a row's entries
// together, so the indexes stream (one thread a row: 141 us for 22M entries
// in 1M rows, its loads a cache line apart; so: 62 us); a wave walks ROWS
// rows, four at a time.
template <int ROWS>
__global__ void __launch_bounds__(256) k_csr_check(int64_t n, int d, int64_t nnz, const int64_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ idx, int bit, int* bad) {
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int64_t base = (blockIdx.x * 4ll + (threadIdx.x >> 6)) * ROWS;
  bool ok = true;
#pragma unroll 4
  for (int q = 0; q < ROWS; q += 4) {
    const int64_t i = base + q + g;
    if (i >= n) break;
    const int64_t p0 = ptr[i], p1 = ptr[i + 1];
    if (p0 >= 0 && p0 <= p1 && p1 <= nnz && (i != 0 || p0 == 0) && (i != n - 1 || p1 == nnz)) {
      int64_t e = p0 + c;
      if constexpr (ROWS < 64)
        for (; e + 112 < p1; e += 128) {   // a long row: sixteen loads in flight
          int j[8], prev[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            j[u] = idx[e + 16 * u];
            prev[u] = idx[max(p0, e + 16 * u - 1)];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if ((e + 16 * u > p0 && j[u] <= prev[u]) || j[u] < 0 || j[u] >= d) ok = false;
        }
      for (; e < p1; e += 16) {
        const int j = idx[e];
        const int prev = e > p0 ? idx[e - 1] : -1;
        if (j <= prev || j < 0 || j >= d) ok = false;
      }
    } else {
      ok = false;
    }
  }
  if (!ok) atomicOr(bad, bit);
}

// A malformed matrix sets `bit` in *bad.  A wave takes 64 rows, 16 or 4: no
// more than have some 1400 entries together, and than leave four waves to every
// SIMD (a CountSketch of 1000 rows of 4000 entries with 64 rows a wave, 16 waves
// in serial loads: 1430 us a call; so 207).
int csr_validate(const CsrView& A, int bit, int* bad, hipStream_t st) {
  auto launch = [&](auto rows_) -> int {
    constexpr int ROWS = decltype(rows_)::value;
    const unsigned blocks = (unsigned)((A.n + 4 * ROWS - 1) / (4 * ROWS));
    hipLaunchKernelGGL((k_csr_check<ROWS>), dim3(blocks), dim3(256), 0, st, A.n, A.d, A.nnz, A.ptr, A.idx, bit, bad);
    SRP_LAUNCH_CHECK();
    return SRP_OK;
  };
  const int64_t rows = std::min<int64_t>(1408 * A.n / std::max<int64_t>(1, A.nnz), A.n / (16ll * num_cus()));
  if (rows >= 64) return launch(std::integral_constant<int, 64>{});
  if (rows >= 16) return launch(std::integral_constant<int, 16>{});
  return launch(std::integral_constant<int, 4>{});
}

// ------------------------------------------------------- CSC build
__global__ void __launch_bounds__(256) k_csc_chunk_count(int64_t n, int d, int chunk_rows,
                                                         const int64_t* __restrict__ ptr,
                                                         const int32_t* __restrict__ idx, int* chunk_cnt) {
  extern __shared__ int cnt[];
  const int ch = blockIdx.x;
  for (int j = threadIdx.x; j < d; j += blockDim.x) cnt[j] = 0;
  __syncthreads();
  const int64_t r0 = (int64_t)ch * chunk_rows, r1 = min(n, r0 + chunk_rows);
  const int64_t e0 = ptr[r0], e1 = ptr[r1];
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) atomicAdd(&cnt[idx[e]], 1);
  __syncthreads();
  for (int j = threadIdx.x; j < d; j += blockDim.x) chunk_cnt[(int64_t)ch * d + j] = cnt[j];
}

// Per column: the chunk counts become offsets inside the column (exclusive
// scan over the chunks, in chunk order); total[j] = entries of column j.
// Three levels over groups of kCscScanGroup chunks: the groups' sums (one
// thread per group and column), their scan per column, then each group's
// chunks from its offset; every level keeps sixteen loads in flight.
constexpr int kCscScanGroup = 64;

__global__ void k_csc_group_sums(int nchunks, int d, const int* __restrict__ chunk_cnt, int* __restrict__ gsum) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int ngroups = (nchunks + kCscScanGroup - 1) / kCscScanGroup;
  if (t >= (int64_t)ngroups * d) return;
  const int g = (int)(t / d), j = (int)(t - (int64_t)g * d);
  const int c0 = g * kCscScanGroup, c1 = min(nchunks, c0 + kCscScanGroup);
  int sum = 0;
  for (int ch0 = c0; ch0 < c1; ch0 += 16) {
    int v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = ch0 + u < c1 ? chunk_cnt[(int64_t)(ch0 + u) * d + j] : 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) sum += v[u];
  }
  gsum[t] = sum;
}

__global__ void k_csc_group_scan(int ngroups, int d, int* __restrict__ gsum, int* __restrict__ total) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d) return;
  int run = 0;
  for (int g0 = 0; g0 < ngroups; g0 += 16) {
    int v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = g0 + u < ngroups ? gsum[(int64_t)(g0 + u) * d + j] : 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (g0 + u < ngroups) gsum[(int64_t)(g0 + u) * d + j] = run;
      run += v[u];
    }
  }
  total[j] = run;
}

__global__ void k_csc_chunk_offsets(int nchunks, int d, const int* __restrict__ gsum, int* __restrict__ chunk_cnt) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int ngroups = (nchunks + kCscScanGroup - 1) / kCscScanGroup;
  if (t >= (int64_t)ngroups * d) return;
  const int g = (int)(t / d), j = (int)(t - (int64_t)g * d);
  const int c0 = g * kCscScanGroup, c1 = min(nchunks, c0 + kCscScanGroup);
  int run = gsum[t];
  for (int ch0 = c0; ch0 < c1; ch0 += 16) {
    int v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = ch0 + u < c1 ? chunk_cnt[(int64_t)(ch0 + u) * d + j] : 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (ch0 + u < c1) chunk_cnt[(int64_t)(ch0 + u) * d + j] = run;
      run += v[u];
    }
  }
}

// One wave per chunk of rows, in row order: the entries of one row have
// distinct columns, so its lanes bump distinct counters; the barrier after
// each row orders the rows.  The chunk's row pointers are staged in LDS
// first, so a row waits only for its own entries.
template <class T>
__global__ void __launch_bounds__(64) k_csc_place(int64_t n, int d, int chunk_rows, const int64_t* __restrict__ ptr,
                                                  const int32_t* __restrict__ idx, const T* __restrict__ val,
                                                  const int* __restrict__ colptr, const int* __restrict__ chunk_off,
                                                  int32_t* __restrict__ rows_out, T* __restrict__ val_out) {
  extern __shared__ int off[];
  int64_t* rp = reinterpret_cast<int64_t*>(off + ((d + 1) & ~1));   // chunk_rows + 1 row pointers
  const int ch = blockIdx.x;
  const int64_t r0 = (int64_t)ch * chunk_rows, r1 = min(n, r0 + chunk_rows);
  for (int j = threadIdx.x; j < d; j += 64) off[j] = colptr[j] + chunk_off[(int64_t)ch * d + j];
  for (int64_t r = r0 + threadIdx.x; r <= r1; r += 64) rp[r - r0] = ptr[r];
  __syncthreads();
  int64_t e0 = rp[0];
  for (int64_t r = r0; r < r1; ++r) {
    const int64_t e1 = rp[r + 1 - r0];
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 64) {
      const int j = idx[e];
      const int pos = off[j];
      off[j] = pos + 1;
      rows_out[pos] = (int32_t)r;
      val_out[pos] = val[e];
    }
    e0 = e1;
    __syncthreads();
  }
}

// Rows per chunk of the CSC build: 128, doubled while the per-chunk column
// counters (chunks x d) would outnumber twice the entries.
static int csc_chunk_rows(int64_t n, int d, int64_t nnz) {
  int rows = 128;
  while (rows < kCscChunkMax && ((n + rows - 1) / rows) * (int64_t)d > 2 * std::max<int64_t>(nnz, 1)) rows *= 2;
  return rows;
}
static int csc_nchunks(const CsrView& A) {
  const int rows = csc_chunk_rows(A.n, A.d, A.nnz);
  return (int)((A.n + rows - 1) / rows);
}

// Segments of kCscSeg entries per column (a column of m entries has
// ceil(m / kCscSeg) of them): at most nnz / kCscSeg + d in all.
int64_t csc_max_segments(const CsrView& A) { return A.nnz / kCscSeg + A.d + 1; }

__global__ void k_csc_seg_count(int d, const int* __restrict__ colptr, int* __restrict__ nseg) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < d) nseg[j] = (colptr[j + 1] - colptr[j] + kCscSeg - 1) / kCscSeg;
}

__global__ void k_csc_seg_fill(int d, const int* __restrict__ segptr, int* __restrict__ segcol) {
  const int j = blockIdx.x;
  for (int q = segptr[j] + threadIdx.x; q < segptr[j + 1]; q += blockDim.x) segcol[q] = j;
}

size_t csc_bytes(const CsrView& A) {
  return 2 * bytes_of<int>((size_t)A.d + 1) + bytes_of<int32_t>((size_t)A.nnz) +
         ((size_t)A.nnz * dtype_size(A.dtype) + 255) / 256 * 256 + bytes_of<int>((size_t)csc_max_segments(A));
}

size_t csc_scratch_bytes(const CsrView& A) {
  const int ngroups = (csc_nchunks(A) + kCscScanGroup - 1) / kCscScanGroup;
  return bytes_of<int>((size_t)csc_nchunks(A) * A.d) + bytes_of<int>((size_t)ngroups * A.d) +
         bytes_of<int>((size_t)A.d + 1);
}

int csc_build(const CsrView& A, CscView* out, Arena& keep, Arena& scratch, hipStream_t st) {
  out->d = A.d;
  out->nnz = A.nnz;
  out->dtype = A.dtype;
  out->ptr = keep.take<int>((size_t)A.d + 1);
  out->idx = keep.take<int32_t>((size_t)A.nnz);
  out->val = keep.take<char>((size_t)A.nnz * dtype_size(A.dtype));
  out->segptr = keep.take<int>((size_t)A.d + 1);
  out->segcol = keep.take<int>((size_t)csc_max_segments(A));
  const int crows = csc_chunk_rows(A.n, A.d, A.nnz);
  const int nch = csc_nchunks(A);
  const int ngroups = (nch + kCscScanGroup - 1) / kCscScanGroup;
  int* chunk = scratch.take<int>((size_t)nch * A.d);
  int* gsum = scratch.take<int>((size_t)ngroups * A.d);
  int* total = scratch.take<int>((size_t)A.d + 1);
  if (!out->segcol || !total) { set_error("CSC copy: workspace too small"); return SRP_ENOMEM; }
  const size_t lds = sizeof(int) * (size_t)A.d;
  const size_t lds_place = sizeof(int) * (size_t)((A.d + 1) & ~1) + sizeof(int64_t) * ((size_t)crows + 1);
  SRP_TRY(allow_dynamic_lds((const void*)k_csc_chunk_count, lds));
  hipLaunchKernelGGL(k_csc_chunk_count, dim3(nch), dim3(256), lds, st, A.n, A.d, crows, A.ptr, A.idx, chunk);
  SRP_LAUNCH_CHECK();
  const unsigned gthreads = (unsigned)(((int64_t)ngroups * A.d + 255) / 256);
  hipLaunchKernelGGL(k_csc_group_sums, dim3(gthreads), dim3(256), 0, st, nch, A.d, chunk, gsum);
  SRP_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_csc_group_scan, dim3((A.d + 255) / 256), dim3(256), 0, st, ngroups, A.d, gsum, total);
  SRP_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_csc_chunk_offsets, dim3(gthreads), dim3(256), 0, st, nch, A.d, gsum, chunk);
  SRP_LAUNCH_CHECK();
  SRP_TRY(scan_excl_i32(total, A.d, out->ptr, st));
  if (A.dtype == SRP_F64) {
    SRP_TRY(allow_dynamic_lds((const void*)k_csc_place<double>, lds_place));
    hipLaunchKernelGGL(k_csc_place<double>, dim3(nch), dim3(64), lds_place, st, A.n, A.d, crows, A.ptr, A.idx,
                       (const double*)A.val, out->ptr, chunk, out->idx, (double*)out->val);
  } else {
    SRP_TRY(allow_dynamic_lds((const void*)k_csc_place<float>, lds_place));
    hipLaunchKernelGGL(k_csc_place<float>, dim3(nch), dim3(64), lds_place, st, A.n, A.d, crows, A.ptr, A.idx,
                       (const float*)A.val, out->ptr, chunk, out->idx, (float*)out->val);
  }
  SRP_LAUNCH_CHECK();
  // segment tables; the segment count is read back once (it sizes the
  // product launches)
  hipLaunchKernelGGL(k_csc_seg_count, dim3((A.d + 255) / 256), dim3(256), 0, st, A.d, out->ptr, total);
  SRP_LAUNCH_CHECK();
  SRP_TRY(scan_excl_i32(total, A.d, out->segptr, st));
  hipLaunchKernelGGL(k_csc_seg_fill, dim3(A.d), dim3(64), 0, st, A.d, out->segptr, out->segcol);
  SRP_LAUNCH_CHECK();
  int nseg = 0;
  SRP_HIP(hipMemcpyAsync(&nseg, out->segptr + A.d, sizeof(int), hipMemcpyDeviceToHost, st));
  SRP_HIP(hipStreamSynchronize(st));
  out->nseg = nseg;
  return SRP_OK;
}

// ------------------------------------------- sparse rows times dense
// Sum of val[e] * D[idx[e]][c] over the entries e0 <= e < e1 (in stored
// order) for lane c of a group of G lanes: the group loads G entries at a
// time (coalesced), broadcasts them by shuffle, and issues the G gathers
// of D before the G multiply-adds, so the gathers are in flight together.
template <class T, int G>
__device__ __forceinline__ double seg_dot(int64_t e0, int64_t e1, const int32_t* __restrict__ idx,
                                          const T* __restrict__ val, const double* __restrict__ D, int ldd, int w,
                                          int c) {
  double acc = 0.0;
  for (int64_t b = e0; b < e1; b += G) {
    const int64_t e = b + c;
    int j = 0;
    double v = 0.0;
    if (e < e1) {
      j = idx[e];
      v = to_f64(val[e]);
    }
    const int m = (int)min<int64_t>(G, e1 - b);
    double dv[G];
#pragma unroll
    for (int t = 0; t < G; ++t) {
      const int jt = __shfl(j, t, G);
      dv[t] = (t < m && c < w) ? D[(int64_t)jt * ldd + c] : 0.0;
    }
#pragma unroll
    for (int t = 0; t < G; ++t) {
      const double vt = __shfl(v, t, G);
      if (t < m) acc += vt * dv[t];
    }
  }
  return acc;
}

// CSR rows: out[r][c] = sum over row r's entries of val[e] * D[idx[e]][c]
// (c < w), minus sub[labels[r]][c] when labels is set.  A group of G lanes
// owns one row.
template <class T, int G>
__global__ void __launch_bounds__(256) k_spmm_rows(int64_t rows, const int64_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ idx, const T* __restrict__ val,
                                                   const double* __restrict__ D, int ldd, int w,
                                                   double* __restrict__ out, int ldo, const double* __restrict__ sub,
                                                   const int32_t* __restrict__ labels, const int* __restrict__ done) {
  if (done && *done) return;
  const int lane = threadIdx.x & 63, g = lane / G, c = lane % G;
  const int64_t r = ((int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64) * (64 / G) + g;
  if (r >= rows) return;   // uniform over the group: shuffles stay inside active groups
  double acc = seg_dot<T, G>(ptr[r], ptr[r + 1], idx, val, D, ldd, w, c);
  if (c < w) {
    if (labels) acc -= sub[(int64_t)labels[r] * w + c];
    out[r * ldo + c] = acc;
  }
}

// CSC columns, stage 1: segment q (kCscSeg entries of column segcol[q] at
// most) gives partial[q][c].
template <class T, int G>
__global__ void __launch_bounds__(256) k_spmm_segs(int nseg, const int* __restrict__ colptr,
                                                   const int* __restrict__ segptr, const int* __restrict__ segcol,
                                                   const int32_t* __restrict__ idx, const T* __restrict__ val,
                                                   const double* __restrict__ D, int ldd, int w,
                                                   double* __restrict__ partial, const int* __restrict__ done) {
  if (done && *done) return;
  const int lane = threadIdx.x & 63, g = lane / G, c = lane % G;
  const int64_t q = ((int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64) * (64 / G) + g;
  if (q >= nseg) return;
  const int j = segcol[q];
  const int64_t e0 = colptr[j] + (int64_t)(q - segptr[j]) * kCscSeg;
  const int64_t e1 = min<int64_t>(colptr[j + 1], e0 + kCscSeg);
  const double acc = seg_dot<T, G>(e0, e1, idx, val, D, ldd, w, c);
  if (c < w) partial[q * w + c] = acc;
}

// Stage 2: out[j][c] = sum of column j's segment partials.  One workgroup
// per column: W lanes per slice (W >= w), 256 / W slices; slice l adds
// segments l, l + 256/W, ... in order, then slice 0 adds the slices'
// sums in slice order (a fixed order: bitwise reproducible).
template <int W>
__global__ void __launch_bounds__(256) k_spmm_seg_sum(int w, const int* __restrict__ segptr,
                                                      const double* __restrict__ partial, double* __restrict__ out,
                                                      int ldo, const int* __restrict__ done) {
  if (done && *done) return;
  constexpr int SL = 256 / W;
  __shared__ double red[SL][W];
  const int j = blockIdx.x, c = threadIdx.x % W, l = threadIdx.x / W;
  double acc = 0.0;
  if (c < w)
    for (int q = segptr[j] + l; q < segptr[j + 1]; q += SL) acc += partial[(int64_t)q * w + c];
  red[l][c] = acc;
  __syncthreads();
  if (l == 0 && c < w) {
    double s = 0.0;
    for (int t = 0; t < SL; ++t) s += red[t][c];
    out[(int64_t)j * ldo + c] = s;
  }
}

// The same products with D in LDS (d x w doubles, the row pitch rounded up
// to a pair of columns): L lanes take a row, two columns each, and walk its
// entries four at a time in stored order.  An entry costs one 16-byte LDS
// read a lane; k_spmm_rows gathers D through the vector cache and broadcasts
// each entry by three lane shuffles (175 us for 22M entries in 1M rows, 8
// columns; so: 108 us,
// bound by the LDS reads).
template <class T> struct SpVec4;
template <> struct SpVec4<float> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct SpVec4<double> { typedef double type __attribute__((ext_vector_type(4), aligned(8))); };
typedef int32_t sp_i32x4 __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kRowsThreads = 1024;

template <class T, int L>
__global__ void __launch_bounds__(kRowsThreads) k_spmm_rows_lds(int64_t rows, int64_t nnz, int d,
                                                               const int64_t* __restrict__ ptr,
                                                               const int32_t* __restrict__ idx,
                                                               const T* __restrict__ val,
                                                               const double* __restrict__ D, int ldd, int w,
                                                               double* __restrict__ out, int ldo,
                                                               const double* __restrict__ sub,
                                                               const int32_t* __restrict__ labels,
                                                               const int* __restrict__ done) {
  if (done && *done) return;
  extern __shared__ double dl[];
  const int wp = (w + 1) & ~1;
  for (int e = threadIdx.x; e < d * wp; e += kRowsThreads) {
    const int j = e / wp, c = e - j * wp;
    dl[e] = c < w ? D[(int64_t)j * ldd + c] : 0.0;
  }
  __syncthreads();
  const int c = threadIdx.x % L;
  const bool on = 2 * c < w;
  const double* dc = dl + (on ? 2 * c : 0);
  auto load = [&](int64_t e, sp_i32x4& j, typename SpVec4<T>::type& v) __attribute__((always_inline)) {
    if (e + 4 <= nnz) {
      j = *reinterpret_cast<const sp_i32x4*>(idx + e);
      v = *reinterpret_cast<const typename SpVec4<T>::type*>(val + e);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        j[t] = e + t < nnz ? idx[e + t] : 0;
        v[t] = e + t < nnz ? val[e + t] : T(0);
      }
    }
  };
  constexpr int RPB = kRowsThreads / L;
  for (int64_t r = blockIdx.x * (int64_t)RPB + threadIdx.x / L; r < rows; r += (int64_t)gridDim.x * RPB) {
    const int64_t p0 = ptr[r], p1 = ptr[r + 1];
    double a0 = 0.0, a1 = 0.0;
    sp_i32x4 j, jn;
    typename SpVec4<T>::type v, vn;
    if (p0 < p1) load(p0, j, v);
    for (int64_t e = p0; e < p1; e += 4) {
      if (e + 4 < p1) load(e + 4, jn, vn);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (e + t < p1) {
          const double2 q = *reinterpret_cast<const double2*>(dc + j[t] * wp);
          const double vt = to_f64((T)v[t]);
          a0 += vt * q.x;
          a1 += vt * q.y;
        }
      j = jn;
      v = vn;
    }
    if (on) {
      if (labels) {
        a0 -= sub[(int64_t)labels[r] * w + 2 * c];
        if (2 * c + 1 < w) a1 -= sub[(int64_t)labels[r] * w + 2 * c + 1];
      }
      out[r * ldo + 2 * c] = a0;
      if (2 * c + 1 < w) out[r * ldo + 2 * c + 1] = a1;
    }
  }
}

// ------------------------------------- transposed products from the rows
// out (d x w) = A^T P without a column copy.  A workgroup takes blocks of at
// most kTsRows rows (and kTsEntries entries), sorts a block's entries by
// column in LDS and then gathers: a group of L lanes owns NC columns of A,
// two P columns a lane, and adds a column's entries in row order to its
// registers, P's rows of the block read from LDS.  The sort is a counting
// sort that needs no order among the threads: each entry sets its row's bit
// in its column's masks, the masks' bit counts scanned over the columns are
// the offsets, and an entry's place is its column's offset plus the bits
// below its own.  Every sum is in a fixed order (rows ascending inside a
// workgroup's range, then the ranges in order), so the result is the same
// bit for bit every time.
//
// Entries and P stream once up to 16 columns of P; past that the blocks are
// sorted again for every 16.  22M entries in 1M rows, 1000 columns, 16
// columns of P: 347 us and 13 for the ranges' sums, bound by the issue of the
// gather's instructions and the LDS latency of its short column runs.  The
// column copy it replaces takes 1053 us to place, then 466 us of 128-byte
// gathers of P at the last-level cache's rate and 62 us of sums; adding row
// after row into LDS sums takes 792 us (random FP64 LDS adds, about 29
// cycles for 44 lanes), one P column a lane instead of two 590 us.
// Taken up to kTsMaxCols columns, where the masks and two columns' sums a lane still
// fit, by the rule of csr_rows_pay; other matrices go through the copy.
constexpr int kTsMaxCols = 2048;
constexpr int kTsThreads = 512;
constexpr int kTsRows = 128;
constexpr int kTsEntries = 4096;   // at least one row of any matrix taken
static_assert(kTsEntries >= kTsMaxCols && kTsRows == 128, "a row fits; four mask words a column");

// A sorted entry: its value and its row in the block.
template <class T> struct TsEntry;
template <> struct alignas(8) TsEntry<float> { float v; int row; };
template <> struct alignas(16) TsEntry<double> { double v; int row; };

template <class T>
static size_t ts_lds(int d, int GL) {
  return (size_t)kTsRows * GL * 8 + (size_t)kTsEntries * sizeof(TsEntry<T>) + (size_t)d * 16 +
         (size_t)(d + 1 + kTsRows + 1 + 8) * 4;
}

// First row of range q of G: ranges of equal weight, an entry counting 1
// and a row 8.
__device__ __forceinline__ int64_t ts_row(int64_t n, int64_t nnz, const int64_t* __restrict__ ptr, int q, int G,
                                          int lane) {
  if (q <= 0) return 0;
  if (q >= G) return n;
  const int64_t target = (int64_t)((double)(nnz + 8 * n) * q / G);
  // smallest r with ptr[r] + 8 r >= target: lo <= r <= hi, 64 probes a step
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t r = min(hi, lo + step * (int64_t)lane);   // lane 0 probes lo
    const int k = __popcll(__ballot(ptr[r] + 8 * r < target));   // probes below the target: a prefix
    if (k == 0) return lo;
    if (k < 64) hi = min(hi, lo + step * (int64_t)k);
    lo = min(hi, lo + step * (int64_t)(k - 1) + 1);
  }
  return lo;
}

template <class T, int L, int NC>
__global__ void __launch_bounds__(kTsThreads, NC <= 16 ? 4 : 2) k_csr_tsum(int64_t n, int d, int64_t nnz,
                                                         const int64_t* __restrict__ ptr,
                                                         const int32_t* __restrict__ idx, const T* __restrict__ val,
                                                         const double* __restrict__ P, int ldp, int w, int G,
                                                         double* __restrict__ partial, const int* __restrict__ done) {
  if (done && *done) return;
  constexpr int RB = kTsRows, NT = kTsThreads, NGR = NT / L, GL = 2 * L;
  extern __shared__ double ts_smem[];
  double* pl = ts_smem;                                    // [RB][GL] rows of P
  TsEntry<T>* ent = reinterpret_cast<TsEntry<T>*>(pl + RB * GL);     // entries by column, then row
  uint32_t* mask = reinterpret_cast<uint32_t*>(ent + kTsEntries);    // [4][d] row bits
  int* off = reinterpret_cast<int*>(mask + 4 * d);         // [d + 1]
  int* pt = off + d + 1;                                   // [RB + 1] row starts
  int* wsum = pt + RB + 1;                                 // [8]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int w0 = blockIdx.y * GL, wt = min(GL, w - w0);
  const int64_t r0 = ts_row(n, nnz, ptr, blockIdx.x, G, lane), r1 = ts_row(n, nnz, ptr, blockIdx.x + 1, G, lane);
  double2 acc[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) acc[i] = make_double2(0.0, 0.0);
  const int g = tid / L, c = 2 * (tid % L);  // gather: column group, first P column
  const int g16 = tid >> 4, l16 = tid & 15; // sort: sixteen lanes a row
  int64_t e0 = ptr[r0];                                           // the block's first entry
  int64_t nptr = r0 < r1 ? ptr[min(r0 + min(tid, RB), r1)] : 0;   // the next block's row starts
  for (int64_t rb = r0; rb < r1;) {
    int nr = (int)min<int64_t>(RB, r1 - rb);
    if (tid <= nr) pt[tid] = (int)(nptr - e0);
    for (int q = tid; q < 4 * d; q += NT) mask[q] = 0;
    __syncthreads();
    // the rows of the block: those that end within kTsEntries (pt ascends)
    nr = __popcll(__ballot(lane < nr && pt[min(lane, nr - 1) + 1] <= kTsEntries)) +
         __popcll(__ballot(lane + 64 < nr && pt[min(lane + 64, nr - 1) + 1] <= kTsEntries));
    const int ne = pt[nr];
    const int32_t* __restrict__ ib = idx + e0;
    const T* __restrict__ vb = val + e0;
    // sixteen lanes a row, four rows each: the first 32 entries of a row are
    // loaded together and stay in registers, the rest follow one by one
    constexpr int RS = RB / (NT / 16);
    int jj[RS][2];
    T vv[RS][2];
    bool in[RS][2];
#pragma unroll
    for (int a = 0; a < RS; ++a)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = g16 + a * (NT / 16), rc = min(r, nr - 1), q = pt[rc] + l16 + 16 * h;
        in[a][h] = r < nr && q < pt[rc + 1];
        const int qc = in[a][h] ? q : 0;
        jj[a][h] = ne > 0 ? ib[qc] : 0;
        vv[a][h] = ne > 0 ? vb[qc] : T(0);
      }
    for (int q = tid; q < nr * GL; q += NT) {
      const int r = q / GL, pc = q % GL;
      pl[q] = pc < wt ? P[(rb + r) * ldp + w0 + pc] : 0.0;
    }
#pragma unroll
    for (int a = 0; a < RS; ++a) {
      const int r = g16 + a * (NT / 16), base = (r >> 5) * d;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (in[a][h]) atomicOr(&mask[base + jj[a][h]], 1u << (r & 31));
      if (r < nr)
        for (int q = pt[r] + l16 + 32; q < pt[r + 1]; q += 16) atomicOr(&mask[base + ib[q]], 1u << (r & 31));
    }
    __syncthreads();
    {   // off = exclusive scan of the columns' counts
      const int per = (d + NT - 1) / NT, j0 = min(d, tid * per), j1 = min(d, j0 + per);
      int sum = 0;
      for (int j = j0; j < j1; ++j)
        sum += __popc(mask[j]) + __popc(mask[d + j]) + __popc(mask[2 * d + j]) + __popc(mask[3 * d + j]);
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
      }
      if (lane == 63) wsum[wv] = incl;
      __syncthreads();
      int run = incl - sum;
      for (int k = 0; k < wv; ++k) run += wsum[k];
      for (int j = j0; j < j1; ++j) {
        off[j] = run;
        run += __popc(mask[j]) + __popc(mask[d + j]) + __popc(mask[2 * d + j]) + __popc(mask[3 * d + j]);
      }
      if (tid == NT - 1) off[d] = run;
    }
    __syncthreads();
    auto place = [&](int r, int j, T v) __attribute__((always_inline)) {
      const int wd = r >> 5;
      int pos = off[j] + __popc(mask[wd * d + j] & ((1u << (r & 31)) - 1u));
      for (int k = 0; k < wd; ++k) pos += __popc(mask[k * d + j]);
      ent[pos] = TsEntry<T>{v, r};
    };
#pragma unroll
    for (int a = 0; a < RS; ++a) {
      const int r = g16 + a * (NT / 16);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (in[a][h]) place(r, jj[a][h], vv[a][h]);
      if (r < nr)
        for (int q = pt[r] + l16 + 32; q < pt[r + 1]; q += 16) place(r, ib[q], vb[q]);
    }
    rb += nr;
    e0 += ne;
    nptr = ptr[min(rb + min(tid, RB), r1)];
    __syncthreads();
    // Four columns of the group at a time: first the columns with more than
    // four entries left, four entries at a time, then an entry of each.
    // Reads past a column's entries take its first place and are not added.
#pragma unroll
    for (int i = 0; i < NC; i += 4) {
      int q0[4], q1[4], most = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = (i + u) * NGR + g;
        q0[u] = j < d ? off[j] : 0;
        q1[u] = j < d ? off[j + 1] : 0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        for (; q1[u] - q0[u] > 4; q0[u] += 4) {
          TsEntry<T> t[4];
          double2 p[4];
#pragma unroll
          for (int h = 0; h < 4; ++h) t[h] = ent[q0[u] + h];
#pragma unroll
          for (int h = 0; h < 4; ++h) p[h] = *reinterpret_cast<const double2*>(&pl[t[h].row * GL + c]);
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            acc[i + u].x = fma(to_f64(t[h].v), p[h].x, acc[i + u].x);
            acc[i + u].y = fma(to_f64(t[h].v), p[h].y, acc[i + u].y);
          }
        }
        most = max(most, q1[u] - q0[u]);
      }
      for (int s = 0; s < most; ++s) {
        TsEntry<T> t[4];
        double2 p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = ent[q0[u] + s < q1[u] ? q0[u] + s : 0];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          p[u] = *reinterpret_cast<const double2*>(&pl[(q0[u] + s < q1[u] ? t[u].row : 0) * GL + c]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (q0[u] + s < q1[u]) {
            acc[i + u].x = fma(to_f64(t[u].v), p[u].x, acc[i + u].x);
            acc[i + u].y = fma(to_f64(t[u].v), p[u].y, acc[i + u].y);
          }
      }
    }
    __syncthreads();
  }
  double* out = partial + ((int64_t)blockIdx.y * G + blockIdx.x) * d * GL;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int j = i * NGR + g;
    if (j < d) *reinterpret_cast<double2*>(&out[(int64_t)j * GL + c]) = acc[i];
  }
}

// out[j][GL y + c] = the ranges' sums in range order: four groups of threads
// take a quarter of the ranges each, sixteen loads in flight, then the
// quarters are added.
__global__ void __launch_bounds__(256) k_csr_tsum_add(const double* __restrict__ partial, int G, int GL, int d, int w,
                                                      double* __restrict__ out, int ldo,
                                                      const int* __restrict__ done) {
  if (done && *done) return;
  __shared__ double q4[4][64];
  const int grp = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t count = (int64_t)d * GL, i = blockIdx.x * 64ll + l;
  const double* part = partial + (int64_t)blockIdx.y * G * count;
  const int per = (G + 3) / 4, z0 = min(G, grp * per), z1 = min(G, z0 + per);
  double v = 0.0;
  if (i < count) {
    int z = z0;
    for (; z + 16 <= z1; z += 16) {
      double t[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) t[u] = part[(z + u) * count + i];
#pragma unroll
      for (int u = 0; u < 16; ++u) v += t[u];
    }
    for (; z < z1; ++z) v += part[z * count + i];
  }
  q4[grp][l] = v;
  __syncthreads();
  if (grp == 0 && i < count) {
    const int64_t j = i / GL;
    const int col = blockIdx.y * GL + (int)(i - j * GL);
    if (col < w) out[j * ldo + col] = ((q4[0][l] + q4[1][l]) + q4[2][l]) + q4[3][l];
  }
}

// P columns of a column group: sixteen at most.
static int ts_lanes(int w) { return w <= 4 ? 4 : w <= 8 ? 8 : 16; }
// Row ranges: two workgroups a CU over all column tiles of P (a range's sums
// are d x 16 doubles of workspace a tile), at least one block of rows or
// entries each (1000 rows of 1000 entries, two matrices, 16 columns of P: in 8
// ranges, a block of rows each, 3406 us a call; in 244 522).
static int ts_ranges(const CsrView& A, int tiles) {
  const int64_t blocks = std::max((A.n + kTsRows - 1) / kTsRows, A.nnz / kTsEntries);
  return (int)std::min(std::max<int64_t>(1, 2ll * num_cus() / tiles), std::max<int64_t>(1, blocks));
}

static bool csr_tsum_ok(const CsrView& A, int w) { return w >= 1 && A.d <= kTsMaxCols; }

// Whether `products` products A^T P (w columns of P) take less time from the
// rows than from the column copy, its build included unless it is there
// anyway.  Both are nearly linear in a few terms; in us, fitted on 64 to 2000
// columns, 1 to 32 entries a row, 66000 to 3M rows, 8 to 64 columns of P:
//  * rows: a block of rows costs 6 to 7.4, its columns (by the columns of P a
//    tile has) and entries more, 1.8 times as much where the sums leave room for
//    one workgroup a CU; the ranges' sums go through memory;
//  * copy: a segment's serial loads, or the gathers of P, a quarter dearer once
//    P is past the caches; the build's fixed cost, a chunk's rows in turn, the
//    chunks' column counts, and placing the entries.
// The rows lose where a block has few entries for each column it looks at:
// 300000 x 1000, 2 entries a row, 32 columns of P: 142 against 35 (the copy
// built in 190); 16 entries, 16 columns 115 and 98; 32 entries 131 and 194; 1M x
// 500, 10 entries, 16 columns 190 and 224 (505).
bool csr_rows_pay(const CsrView& A, int w, int products, bool copy_there) {
  if (!csr_tsum_ok(A, w)) return false;
  const int GL = ts_lanes(w), tiles = (w + GL - 1) / GL, G = ts_ranges(A, tiles);
  const double n = (double)A.n, nnz = (double)A.nnz, x = A.d * GL / 16.0;
  const double blocks = (double)std::max<int64_t>(1, std::max((A.n + kTsRows - 1) / kTsRows, A.nnz / kTsEntries));
  double block = (GL <= 8 ? 6.0 : 7.4) + 0.0045 * std::min(x, 1024.0) + nnz / blocks * (0.001 + 1.5e-6 * x);
  if (x > 1024.0) block *= 1.8;
  const double rows = (blocks / G + 1.0) * block + 5.0 + (double)A.d * GL * G * tiles * 1e-6;
  const double segment = std::min<double>(kCscSeg, nnz / A.d) * (w <= 8 ? 0.14 : 0.1);
  const double far = 1.0 + 0.25 * std::min(1.0, std::max(0.0, (n - 3e5) / 7e5));
  const double copy = 5.0 + std::max(segment, nnz * 1e-6 * (w <= 16 ? 18.0 : 1.1 * w) * far);
  const double build = copy_there ? 0.0
                                  : 130.0 + 0.19 * csc_chunk_rows(A.n, A.d, A.nnz) + 15e-6 * nnz +
                                        30e-6 * std::max(0.0, nnz - 4e6) + 10e-6 * A.d * csc_nchunks(A);
  return products * rows <= products * copy + build;
}

size_t csr_tsum_bytes(const CsrView& A, int w) {
  const int GL = ts_lanes(w), tiles = (w + GL - 1) / GL;
  return bytes_of<double>((size_t)tiles * ts_ranges(A, tiles) * A.d * GL);
}

template <class T, int L>
static int tsum_launch(const CsrView& A, const double* P, int ldp, int w, double* partial, const int* done,
                       hipStream_t st) {
  constexpr int GL = 2 * L;
  const int tiles = (w + GL - 1) / GL, G = ts_ranges(A, tiles);
  const dim3 grid((unsigned)G, (unsigned)tiles);
  const size_t lds = ts_lds<T>(A.d, GL);
  const int nc = (A.d + kTsThreads / L - 1) / (kTsThreads / L);   // columns of A per group
#define SRP_TS_CASE(NC_)                                                                                            \
  if (nc <= NC_) {                                                                                                  \
    SRP_TRY(allow_dynamic_lds((const void*)k_csr_tsum<T, L, NC_>, ts_lds<T>(kTsMaxCols, GL)));                      \
    hipLaunchKernelGGL((k_csr_tsum<T, L, NC_>), grid, dim3(kTsThreads), lds, st, A.n, A.d, A.nnz, A.ptr, A.idx,     \
                       (const T*)A.val, P, ldp, w, G, partial, done);                                               \
    SRP_LAUNCH_CHECK();                                                                                             \
    return SRP_OK;                                                                                                  \
  }
  SRP_TS_CASE(4)
  SRP_TS_CASE(8)
  if constexpr (L >= 4) { SRP_TS_CASE(16) }
  if constexpr (L >= 8) { SRP_TS_CASE(32) }
#undef SRP_TS_CASE
  set_error("sparse transposed product: no instance for %d columns", A.d);
  return SRP_EINVAL;
}

template <class T>
static int tsum_dispatch(const CsrView& A, const double* P, int ldp, int w, double* partial, const int* done,
                         hipStream_t st) {
  switch (ts_lanes(w)) {
    case 4: return tsum_launch<T, 2>(A, P, ldp, w, partial, done, st);
    case 8: return tsum_launch<T, 4>(A, P, ldp, w, partial, done, st);
    default: return tsum_launch<T, 8>(A, P, ldp, w, partial, done, st);
  }
}

int csr_tsum(const CsrView& A, const double* P, int ldp, int w, double* out, int ldo, double* partial,
             const int* done, hipStream_t st) {
  SRP_REQUIRE(csr_tsum_ok(A, w), "sparse product width %d, %d columns", w, A.d);
  if (A.dtype == SRP_F64) SRP_TRY(tsum_dispatch<double>(A, P, ldp, w, partial, done, st));
  else SRP_TRY(tsum_dispatch<float>(A, P, ldp, w, partial, done, st));
  const int GL = ts_lanes(w), tiles = (w + GL - 1) / GL;
  const dim3 grid((unsigned)(((int64_t)A.d * GL + 63) / 64), (unsigned)tiles);
  hipLaunchKernelGGL(k_csr_tsum_add, grid, dim3(256), 0, st, partial, ts_ranges(A, tiles), GL, A.d, w, out, ldo, done);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

// D in LDS while it fits one workgroup a CU (two while it fits half).
constexpr size_t kRowsLds = 150 * 1024;

template <class T, int L>
static int spmm_rows_lds_launch(const CsrView& A, const T* val, const double* D, int ldd, int w, double* out, int ldo,
                                const double* sub, const int32_t* labels, const int* done, hipStream_t st) {
  const size_t lds = (size_t)A.d * ((w + 1) & ~1) * 8;
  const int per_cu = lds <= 76 * 1024 ? 2 : 1;
  const int64_t rpb = kRowsThreads / L;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((A.n + rpb - 1) / rpb,
                                                                         (int64_t)per_cu * num_cus()));
  SRP_TRY(allow_dynamic_lds((const void*)k_spmm_rows_lds<T, L>, kRowsLds));
  hipLaunchKernelGGL((k_spmm_rows_lds<T, L>), dim3(grid), dim3(kRowsThreads), lds, st, A.n, A.nnz, A.d, A.ptr, A.idx,
                     val, D, ldd, w, out, ldo, sub, labels, done);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

template <class T>
static int spmm_rows_lds(const CsrView& A, const T* val, const double* D, int ldd, int w, double* out, int ldo,
                         const double* sub, const int32_t* labels, const int* done, hipStream_t st) {
  if (w <= 2) return spmm_rows_lds_launch<T, 1>(A, val, D, ldd, w, out, ldo, sub, labels, done, st);
  if (w <= 4) return spmm_rows_lds_launch<T, 2>(A, val, D, ldd, w, out, ldo, sub, labels, done, st);
  if (w <= 8) return spmm_rows_lds_launch<T, 4>(A, val, D, ldd, w, out, ldo, sub, labels, done, st);
  if (w <= 16) return spmm_rows_lds_launch<T, 8>(A, val, D, ldd, w, out, ldo, sub, labels, done, st);
  return spmm_rows_lds_launch<T, 16>(A, val, D, ldd, w, out, ldo, sub, labels, done, st);
}

template <class T>
static int spmm_rows_launch(int64_t rows, const int64_t* ptr, const int32_t* idx, const T* val, const double* D,
                            int ldd, int w, double* out, int ldo, const double* sub, const int32_t* labels,
                            const int* done, hipStream_t st) {
  auto grid = [&](int G) { return dim3((unsigned)((rows + (4 * (64 / G)) - 1) / (4 * (64 / G)))); };
  if (w <= 8) hipLaunchKernelGGL((k_spmm_rows<T, 8>), grid(8), dim3(256), 0, st, rows, ptr, idx, val, D, ldd, w,
                                 out, ldo, sub, labels, done);
  else if (w <= 16) hipLaunchKernelGGL((k_spmm_rows<T, 16>), grid(16), dim3(256), 0, st, rows, ptr, idx, val, D,
                                       ldd, w, out, ldo, sub, labels, done);
  else if (w <= 32) hipLaunchKernelGGL((k_spmm_rows<T, 32>), grid(32), dim3(256), 0, st, rows, ptr, idx, val, D,
                                       ldd, w, out, ldo, sub, labels, done);
  else hipLaunchKernelGGL((k_spmm_rows<T, 64>), grid(64), dim3(256), 0, st, rows, ptr, idx, val, D, ldd, w, out,
                          ldo, sub, labels, done);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

template <class T>
static int spmm_segs_launch(const CscView& A, const T* val, const double* D, int ldd, int w, double* partial,
                            const int* done, hipStream_t st) {
  const int64_t n = A.nseg;
  auto grid = [&](int G) { return dim3((unsigned)((n + (4 * (64 / G)) - 1) / (4 * (64 / G)))); };
  if (w <= 8) hipLaunchKernelGGL((k_spmm_segs<T, 8>), grid(8), dim3(256), 0, st, A.nseg, A.ptr, A.segptr, A.segcol,
                                 A.idx, val, D, ldd, w, partial, done);
  else if (w <= 16) hipLaunchKernelGGL((k_spmm_segs<T, 16>), grid(16), dim3(256), 0, st, A.nseg, A.ptr, A.segptr,
                                       A.segcol, A.idx, val, D, ldd, w, partial, done);
  else if (w <= 32) hipLaunchKernelGGL((k_spmm_segs<T, 32>), grid(32), dim3(256), 0, st, A.nseg, A.ptr, A.segptr,
                                       A.segcol, A.idx, val, D, ldd, w, partial, done);
  else hipLaunchKernelGGL((k_spmm_segs<T, 64>), grid(64), dim3(256), 0, st, A.nseg, A.ptr, A.segptr, A.segcol,
                          A.idx, val, D, ldd, w, partial, done);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

int csr_times_dense(const CsrView& A, const double* D, int ldd, int w, double* out, int ldo, const double* sub,
                    const int32_t* labels, const int* done, hipStream_t st) {
  SRP_REQUIRE(w >= 1 && w <= 64, "sparse product width %d outside 1..64", w);
  if (A.n <= 0) return SRP_OK;
  // D in LDS pays once the rows fill a workgroup of it on every CU (below,
  // the gathers' four times smaller workgroups spread the rows better)
  const int64_t rpb = kRowsThreads / (w <= 2 ? 1 : w <= 4 ? 2 : w <= 8 ? 4 : w <= 16 ? 8 : 16);
  if (w <= 32 && (size_t)A.d * ((w + 1) & ~1) * 8 <= kRowsLds && A.n >= rpb * num_cus()) {
    if (A.dtype == SRP_F64)
      return spmm_rows_lds(A, (const double*)A.val, D, ldd, w, out, ldo, sub, labels, done, st);
    return spmm_rows_lds(A, (const float*)A.val, D, ldd, w, out, ldo, sub, labels, done, st);
  }
  if (A.dtype == SRP_F64)
    return spmm_rows_launch(A.n, A.ptr, A.idx, (const double*)A.val, D, ldd, w, out, ldo, sub, labels, done, st);
  return spmm_rows_launch(A.n, A.ptr, A.idx, (const float*)A.val, D, ldd, w, out, ldo, sub, labels, done, st);
}

size_t csc_partial_bytes(const CsrView& A, int w) {
  return bytes_of<double>((size_t)csc_max_segments(A) * w);
}

int csc_times_dense(const CscView& A, const double* D, int ldd, int w, double* out, int ldo, double* partial,
                    const int* done, hipStream_t st) {
  SRP_REQUIRE(w >= 1 && w <= 64, "sparse product width %d outside 1..64", w);
  if (A.d <= 0) return SRP_OK;
  if (A.nseg > 0) {
    if (A.dtype == SRP_F64) SRP_TRY(spmm_segs_launch(A, (const double*)A.val, D, ldd, w, partial, done, st));
    else SRP_TRY(spmm_segs_launch(A, (const float*)A.val, D, ldd, w, partial, done, st));
  }
  if (w <= 8) hipLaunchKernelGGL(k_spmm_seg_sum<8>, dim3(A.d), dim3(256), 0, st, w, A.segptr, partial, out, ldo, done);
  else if (w <= 16) hipLaunchKernelGGL(k_spmm_seg_sum<16>, dim3(A.d), dim3(256), 0, st, w, A.segptr, partial, out, ldo,
                                       done);
  else if (w <= 32) hipLaunchKernelGGL(k_spmm_seg_sum<32>, dim3(A.d), dim3(256), 0, st, w, A.segptr, partial, out, ldo,
                                       done);
  else hipLaunchKernelGGL(k_spmm_seg_sum<64>, dim3(A.d), dim3(256), 0, st, w, A.segptr, partial, out, ldo, done);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

// ------------------------------------------------- CSR CountSketch
// One workgroup per bucket; its rows (ascending) are added into an LDS row
// of d doubles, one row at a time (a row's columns are distinct, so its
// threads write distinct words; the barrier orders the rows).  With labels,
// the bucket's signed class counts (S E for the one-hot E) ride along.
template <class T>
__global__ void __launch_bounds__(256) k_cs_csr(int d, uint64_t seed, const int* __restrict__ offsets,
                                                const int* __restrict__ sorted, const int64_t* __restrict__ ptr,
                                                const int32_t* __restrict__ idx, const T* __restrict__ val,
                                                double* __restrict__ out, const int32_t* __restrict__ labels, int c,
                                                double* __restrict__ se) {
  extern __shared__ double acc[];
  const int b = blockIdx.x;
  const int w = d + (labels ? c : 0);
  for (int j = threadIdx.x; j < w; j += blockDim.x) acc[j] = 0.0;
  __syncthreads();
  const int beg = offsets[b], cnt = offsets[b + 1] - beg;
  for (int q = 0; q < cnt; ++q) {
    const int row = sorted[beg + q];
    const double g = (double)cs_sign(splitmix64(seed, (uint64_t)row));
    const int64_t e0 = ptr[row], e1 = ptr[row + 1];
    for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) acc[idx[e]] += g * to_f64(val[e]);
    if (labels && threadIdx.x == 0) acc[d + labels[row]] += g;
    __syncthreads();
  }
  for (int j = threadIdx.x; j < d; j += blockDim.x) out[(int64_t)b * d + j] = acc[j];
  if (labels)
    for (int j = threadIdx.x; j < c; j += blockDim.x) se[(int64_t)b * c + j] = acc[d + j];
}

size_t countsketch_csr_ws_bytes(int64_t n, int s) { return countsketch_ws_bytes(n, s); }

int countsketch_csr_run(const CsrView& A, int s, uint64_t seed, double* out, const int32_t* labels, int c,
                        double* se, Arena& ws, hipStream_t st) {
  SRP_REQUIRE(A.d <= kCsrMaxCols, "CSR input wider than %d columns", kCsrMaxCols);
  const int* offsets = nullptr;
  const int* sorted = nullptr;
  SRP_TRY(countsketch_buckets(A.n, s, seed, ws, &offsets, &sorted, st));
  const size_t lds = sizeof(double) * (size_t)(A.d + (labels ? c : 0));
  if (A.dtype == SRP_F64) {
    SRP_TRY(allow_dynamic_lds((const void*)k_cs_csr<double>, lds));
    hipLaunchKernelGGL(k_cs_csr<double>, dim3(s), dim3(256), lds, st, A.d, seed, offsets, sorted, A.ptr, A.idx,
                       (const double*)A.val, out, labels, c, se);
  } else {
    SRP_TRY(allow_dynamic_lds((const void*)k_cs_csr<float>, lds));
    hipLaunchKernelGGL(k_cs_csr<float>, dim3(s), dim3(256), lds, st, A.d, seed, offsets, sorted, A.ptr, A.idx,
                       (const float*)A.val, out, labels, c, se);
  }
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

// ------------------------------------------------- FDA class statistics
__global__ void __launch_bounds__(256) k_label_counts(int64_t n, int c, const int32_t* __restrict__ labels,
                                                      int* counts, int* bad) {
  __shared__ int h[kLdaMaxClasses];
  for (int q = threadIdx.x; q < c; q += blockDim.x) h[q] = 0;
  __syncthreads();
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) {
    const int y = labels[i];
    if (y < 0 || y >= c) atomicOr(bad, 1);
    else atomicAdd(&h[y], 1);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < c; q += blockDim.x)
    if (h[q]) atomicAdd(&counts[q], h[q]);
}

int label_counts_run(int64_t n, int c, const int32_t* labels, int* counts, int* bad, hipStream_t st) {
  SRP_TRY(fill_i32(counts, c, 0, st));
  hipLaunchKernelGGL(k_label_counts, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, c, labels, counts, bad);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

// Class sums of column j: one wave per column, lane l adds the column's
// entries l, l + 64, ... into its own LDS slot per class, then the slots
// are summed in lane order.  Labels must already be known to be in range.
template <class T>
__global__ void __launch_bounds__(64) k_csc_class_sums(int d, int c, const int* __restrict__ colptr,
                                                       const int32_t* __restrict__ rows, const T* __restrict__ val,
                                                       const int32_t* __restrict__ labels, double* __restrict__ sums) {
  __shared__ double acc[kLdaMaxClasses * 64];
  const int j = blockIdx.x, lane = threadIdx.x;
  for (int q = 0; q < c; ++q) acc[q * 64 + lane] = 0.0;
  const int e0 = colptr[j], e1 = colptr[j + 1];
  for (int e = e0 + lane; e < e1; e += 64) acc[labels[rows[e]] * 64 + lane] += to_f64(val[e]);
  __syncthreads();
  for (int q = lane; q < c; q += 64) {
    double s = 0.0;
    for (int l = 0; l < 64; ++l) s += acc[q * 64 + l];
    sums[(int64_t)q * d + j] = s;
  }
}

// Per column j: m_q = sums_q / n_q, m = sum_q sums_q / n,
// Yhat_q = sqrt(n_q) (m_q - m).
__global__ void k_fda_class_factors(int64_t n, int d, int c, const int* __restrict__ counts,
                                    const double* __restrict__ sums, double* __restrict__ means,
                                    double* __restrict__ Yhat) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d) return;
  double tot = 0.0;
  for (int q = 0; q < c; ++q) tot += sums[(int64_t)q * d + j];
  const double m = tot / (double)n;
  for (int q = 0; q < c; ++q) {
    const double mq = sums[(int64_t)q * d + j] / (double)counts[q];
    means[(int64_t)q * d + j] = mq;
    Yhat[(int64_t)q * d + j] = sqrt((double)counts[q]) * (mq - m);
  }
}

int fda_csr_stats_run(const CscView& A, int64_t n, int c, const int32_t* labels, const int* counts, double* sums,
                      double* means, double* Yhat, hipStream_t st) {
  if (A.dtype == SRP_F64)
    hipLaunchKernelGGL(k_csc_class_sums<double>, dim3(A.d), dim3(64), 0, st, A.d, c, A.ptr, A.idx,
                       (const double*)A.val, labels, sums);
  else
    hipLaunchKernelGGL(k_csc_class_sums<float>, dim3(A.d), dim3(64), 0, st, A.d, c, A.ptr, A.idx,
                       (const float*)A.val, labels, sums);
  SRP_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_fda_class_factors, dim3((A.d + 255) / 256), dim3(256), 0, st, n, A.d, c, counts, sums, means,
                     Yhat);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

}  // namespace srp

namespace srp {

int csr_check(int count, const CsrView* A, const char* const* names, int* bad, hipStream_t st) {
  SRP_TRY(fill_i32(bad, 1, 0, st));
  for (int q = 0; q < count; ++q) {
    SRP_REQUIRE(A[q].n >= 1 && A[q].n < (int64_t(1) << 31), "%s: rows out of range", names[q]);
    SRP_REQUIRE(A[q].d >= 1 && A[q].d <= kCsrMaxCols, "%s: need 1 <= columns <= %d", names[q], kCsrMaxCols);
    SRP_REQUIRE(A[q].nnz >= 0 && A[q].nnz < (int64_t(1) << 31), "%s: nnz out of range", names[q]);
    SRP_REQUIRE(A[q].dtype == SRP_F32 || A[q].dtype == SRP_F64, "%s: values must be SRP_F32 or SRP_F64", names[q]);
    SRP_REQUIRE(A[q].ptr && (A[q].nnz == 0 || (A[q].idx && A[q].val)), "%s: null pointer", names[q]);
    SRP_TRY(csr_validate(A[q], 1 << q, bad, st));
  }
  int h = 0;
  SRP_HIP(hipMemcpyAsync(&h, bad, sizeof(int), hipMemcpyDeviceToHost, st));
  SRP_HIP(hipStreamSynchronize(st));
  for (int q = 0; q < count; ++q)
    SRP_REQUIRE(!(h >> q & 1), "%s is not a well-formed CSR matrix (row pointers, or columns in range and strictly "
                "increasing)", names[q]);
  return SRP_OK;
}

}  // namespace srp
