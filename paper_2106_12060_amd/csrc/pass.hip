// Fused tall-skinny data pass: for data blocks A_0 (n x d0), A_1 (n x d1)
// and directions W_0, W_1 (d_b x k) compute, in one read of the data,
//     J_b = A_b^T [A_0 W_0 | A_1 W_1]        (d_b x NB k).
// These are the products with the data matrices that every Riemannian
// component of Table 1 needs (X^T X U, X^T Y V, ...; costs in Table costs:
// O(n d p) per product).
//
// Work split: a workgroup of 8 waves streams 16-row blocks of [A_0 | A_1].
// Each row block is handled by a PAIR of workgroups (block indices 8 apart,
// so both run on the same XCD and the second read of the block is served
// by that XCD's L2): both form the full P from their LDS copy, and each
// accumulates A_b^T [P_0 | P_1] for half of the columns, which halves the
// accumulator registers a wave must keep.
// The block is staged in LDS (row-major, row pitch = 4 mod 64 elements so
// both access patterns below are bank-conflict free; A_1's tiles follow
// A_0's, and the columns between a view's last and its last tile's are
// zeros: the tiles there meet zero directions, which an infinity or a NaN of
// another column would survive.  The loads place the columns, past a row's
// end they give zeros: 100000 x (501 + 300) BF16 in FP32 at k = 8 takes 562
// us, 792 where the stores move A_1's columns); while the matrix
// cores work on block i, the global loads of the workgroup's next block are
// already in flight into registers.  The direction operands of a wave's
// P tiles stay in registers for the whole launch when they fit (64 per
// lane); otherwise they are re-read from L2 per block, before the next
// block's loads are issued, so that a wait on them never waits on HBM.  Columns are cut into 16-wide tiles;
// wave w owns tiles w, w+8, ...  For each block a wave
//   (b) accumulates its tiles' share of P_b = A_b W_b (16 x k) on the matrix
//       cores (A-operand lane: row = lane%16, column = 4 step + lane/16),
//   (c) the 8 partial P's are summed through LDS,
//   (d) accumulates its tiles' rows of A_b^T [P_0 | P_1] (A-operand lane:
//       column = lane%16, row = 4 (lane/16) + step).
// Each workgroup keeps its accumulators in registers over all its row
// blocks and writes one partial; a second kernel sums the partials in a
// fixed order (deterministic, no atomics).
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <type_traits>

namespace srp {

constexpr int kPassWaves = 8;
constexpr int kPassThreads = 64 * kPassWaves;
constexpr int kLdsBytes = 160 * 1024;   // of a CU
constexpr int kPassLds = 150 * 1024;    // of the row-block stage for rows of d0 + d1 columns; whole tiles take 8 KB more at most

// Largest d0 + d1 per compute type, and loads per row per thread.
template <class CT> struct PassCfg;
// jpf of the jpr 512-column chunks of a row block are prefetched into
// registers during the previous block's math; the rest load on demand.
template <> struct PassCfg<float> { static constexpr int dmax = 2048; static constexpr int jpr = 4; static constexpr int jpf = 4; };
template <> struct PassCfg<double> { static constexpr int dmax = 896; static constexpr int jpr = 2; static constexpr int jpf = 2; };

__host__ __device__ constexpr int pass_pitch(int D) { return ((D + 63) / 64) * 64 + 4; }

// Pack double d_b x k directions into zero-padded (ceil16(d_b) x kpad) CT
// matrices, both blocks in one launch (block 1 follows block 0's elements).
template <class CT>
__global__ void k_pack_dir(const double* __restrict__ W0, int d0, int dpad0, CT* __restrict__ Wp0,
                           const double* __restrict__ W1, int d1, int dpad1, CT* __restrict__ Wp1, int k, int kpad) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t n0 = (int64_t)dpad0 * kpad;
  const double* W = W0;
  CT* Wp = Wp0;
  int d = d0;
  if (i >= n0) {
    i -= n0;
    if (i >= (int64_t)dpad1 * kpad) return;
    W = W1;
    Wp = Wp1;
    d = d1;
  }
  const int r = (int)(i / kpad), c = (int)(i - (int64_t)r * kpad);
  Wp[i] = (r < d && c < k) ? (CT)W[(int64_t)r * k + c] : CT(0);
}

template <class CT>
static int pack_dirs(const double* W0, int d0, int dp0, CT* Wp0, const double* W1, int d1, int dp1, CT* Wp1, int k,
                     int KP, hipStream_t st) {
  const int64_t tot = (int64_t)dp0 * KP + (Wp1 ? (int64_t)dp1 * KP : 0);
  hipLaunchKernelGGL((k_pack_dir<CT>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, W0, d0, dp0, Wp0, W1,
                     d1, Wp1 ? dp1 : 0, Wp1, k, KP);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

template <class CT, class DT> __device__ __forceinline__ CT cvt(DT v);
template <> __device__ __forceinline__ float cvt<float, float>(float v) { return v; }
template <> __device__ __forceinline__ float cvt<float, bf16>(bf16 v) { return __bfloat162float(v); }
template <> __device__ __forceinline__ double cvt<double, double>(double v) { return v; }
template <> __device__ __forceinline__ double cvt<double, float>(float v) { return (double)v; }
template <> __device__ __forceinline__ double cvt<double, bf16>(bf16 v) { return (double)__bfloat162float(v); }


constexpr int kPassSplit = 2;   // column halves per row block
constexpr int kXcds = 8;

// TMAX: most tiles of [A_0 | A_1] (two views that do not end on tiles take
// one more than their columns alone would).
template <class DT, class CT, int NB, int KT, int TMAX>
__global__ void __launch_bounds__(kPassThreads) k_pass(const DT* __restrict__ A0, const DT* __restrict__ A1,
                                                       int64_t n, int d0, int d1, int k,
                                                       const CT* __restrict__ Wp0, const CT* __restrict__ Wp1,
                                                       int nrb, CT* __restrict__ partial,
                                                       const int* __restrict__ done) {
  if (done && *done) return;
  constexpr int JPR = PassCfg<CT>::jpr;
  constexpr int JPF = PassCfg<CT>::jpf;
  constexpr int TPW = (TMAX + kPassWaves * kPassSplit - 1) / (kPassWaves * kPassSplit);
  constexpr int NT = NB * KT;
  constexpr int KP = KT * 16;
  constexpr int TPB = (TMAX + kPassWaves - 1) / kPassWaves;        // P tiles per wave
  constexpr bool WREG = TPB * 4 * KT * (int)sizeof(CT) <= 64 * 4;       // W operands in registers
  using acc_t = typename Acc4<CT>::type;
  extern __shared__ unsigned char pass_smem[];
  const int D = d0 + (NB == 2 ? d1 : 0);
  const int T0 = (d0 + 15) >> 4;
  const int TT = T0 + (NB == 2 ? ((d1 + 15) >> 4) : 0);
  const int pitch = pass_pitch(16 * TT);
  CT* xs = reinterpret_cast<CT*>(pass_smem);                 // [16][pitch]
  CT* red = xs + 16 * pitch;                                  // [waves][NT][256]
  CT* pfull = red + kPassWaves * NT * 256;                    // [NT][16][17]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  // pair mapping: XCD x, half h, group q  ->  row group rg
  const int bx = blockIdx.x;
  const int xcd = bx % kXcds, half = (bx / kXcds) % kPassSplit, grp = bx / (kXcds * kPassSplit);
  const int rg = grp * kXcds + xcd;
  const int ngroups = gridDim.x / kPassSplit;
  const int TH = (TT + kPassSplit - 1) / kPassSplit;     // tiles per half
  const int tbeg = half * TH, tend = min(TT, tbeg + TH);
  const __amdgpu_buffer_rsrc_t wr0 = make_rsrc(Wp0, (int64_t)((d0 + 15) / 16 * 16) * KP * sizeof(CT));
  const __amdgpu_buffer_rsrc_t wr1 =
      make_rsrc(NB == 2 ? Wp1 : Wp0, (int64_t)((((NB == 2 ? d1 : d0) + 15) / 16) * 16) * KP * sizeof(CT));
  const int wvoff = (g * KP + l16) * (int)sizeof(CT);

  acc_t acc[TPW][NT];
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // direction operands of this wave's P tiles: tile t = w + 8 i, step s2
  CT wreg[WREG ? TPB : 1][4][KT];
  auto w_operand = [&](int t, int s2, int kt) __attribute__((always_inline)) -> CT {
    const bool b1 = (NB == 2) && (t >= T0);
    const int ct = b1 ? t - T0 : t;
    const int soff = ((ct * 16 + 4 * s2) * KP + kt * 16) * (int)sizeof(CT);
    return b1 ? buf_load<CT>(wr1, wvoff + soff, 0) : buf_load<CT>(wr0, wvoff + soff, 0);
  };
  if (WREG) {
#pragma unroll
    for (int i = 0; i < (WREG ? TPB : 1); ++i)
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const int t = w + kPassWaves * i;
          wreg[i][s2][kt] = (t < TT) ? w_operand(t, s2, kt) : CT(0);
        }
  }

  // Row r of the block gets its own buffer resource (scalar), holding
  // exactly the d_b elements of that row, or none past row n; a lane reads
  // column c of the tiles with one lane offset for all rows, and every
  // out-of-row, out-of-block or out-of-matrix element reads as zero: so the
  // columns between a view's last and its last tile's end come as zeros.
  auto row_rsrc = [&](const DT* A, int db, int64_t row) __attribute__((always_inline)) {
    return make_rsrc(A + row * db, row < n ? (int64_t)db * (int64_t)sizeof(DT) : 0);
  };
  auto load_elem = [&](int64_t row, int j) __attribute__((always_inline)) -> DT {
    const int cb = kPassThreads * j;        // uniform chunk start
    const int c = cb + tid;
    const int v0 = c * (int)sizeof(DT);
    if (NB == 1 || cb + kPassThreads <= 16 * T0) return buf_load<DT>(row_rsrc(A0, d0, row), v0, 0);
    const int v1 = (c - 16 * T0) * (int)sizeof(DT);   // negative = out of range
    if (cb >= 16 * T0) return buf_load<DT>(row_rsrc(A1, d1, row), v1, 0);
    const DT x0 = buf_load<DT>(row_rsrc(A0, d0, row), v0, 0);
    const DT x1 = buf_load<DT>(row_rsrc(A1, d1, row), v1, 0);
    return (c < 16 * T0) ? x0 : x1;
  };
  DT pf[16][JPF];
  // the one tile past the chunks (an A_1 that follows an A_0 which does not
  // end on a tile): an element a thread
  constexpr int kChunked = kPassThreads * JPR;
  constexpr bool kTail = 16 * TMAX > kChunked;
  static_assert(16 * TMAX <= kChunked + 16, "one tile past the chunks");
  DT pft{};
  auto prefetch = [&](int rbk) __attribute__((always_inline)) {
    const int64_t r0 = (int64_t)rbk * 16;
#pragma unroll
    for (int j = 0; j < JPF; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) pf[r][j] = load_elem(r0 + r, j);
    if (kTail) {
      const int64_t row = r0 + (tid >> 4);
      const int c = kChunked + (tid & 15) - 16 * T0;
      pft = tid < 256 && row < n && c < d1 ? A1[row * d1 + c] : DT{};
    }
  };

  int rb = rg;
  if (rb < nrb) prefetch(rb);
  for (; rb < nrb; rb += ngroups) {
    __syncthreads();   // previous block fully consumed
#pragma unroll
    for (int j = 0; j < JPF; ++j) {
      const int c = tid + kPassThreads * j;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (c < 16 * TT) xs[r * pitch + c] = cvt<CT>(pf[r][j]);
    }
    if (JPF < JPR) {
#pragma unroll
      for (int j = JPF; j < JPR; ++j) {
        const int c = tid + kPassThreads * j;
        if (kPassThreads * j < 16 * TT) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const DT v = load_elem((int64_t)rb * 16 + r, j);
            if (c < 16 * TT) xs[r * pitch + c] = cvt<CT>(v);
          }
        }
      }
    }
    if (kTail && tid < 256) xs[(tid >> 4) * pitch + kChunked + (tid & 15)] = cvt<CT>(pft);
    __syncthreads();
    if (WREG && rb + ngroups < nrb) prefetch(rb + ngroups);   // in flight during the math
    // (b) P_b partials
    acc_t pacc[NB][KT];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) pacc[b][kt] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < TPB; ++i) {
      const int t = w + kPassWaves * i;
      if (t < TT) {
        const bool b1 = (NB == 2) && (t >= T0);
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
          const CT a = xs[l16 * pitch + 16 * t + 4 * s2 + g];
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            const CT bw = WREG ? wreg[WREG ? i : 0][s2][kt] : w_operand(t, s2, kt);
            if (b1) pacc[NB - 1][kt] = mfma16x16x4(a, bw, pacc[NB - 1][kt]);
            else pacc[0][kt] = mfma16x16x4(a, bw, pacc[0][kt]);
          }
        }
      }
    }
    if (!WREG && rb + ngroups < nrb) prefetch(rb + ngroups);   // in flight during (c), (d)
    // (c) reduce P over waves
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[(w * NT + b * KT + kt) * 256 + acc_row<CT>(lane, r) * 16 + l16] = pacc[b][kt][r];
    __syncthreads();
    for (int e = tid; e < NT * 256; e += kPassThreads) {
      const int nt = e >> 8, q = e & 255;
      CT v = CT(0);
#pragma unroll
      for (int ww = 0; ww < kPassWaves; ++ww) v += red[(ww * NT + nt) * 256 + q];
      pfull[nt * 272 + (q >> 4) * 17 + (q & 15)] = v;
    }
    __syncthreads();
    // (d) A_b^T [P_0 | P_1] for this workgroup's half of the tiles
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int t = tbeg + w + kPassWaves * i;
      if (t < tend) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const CT a = xs[(4 * g + s) * pitch + 16 * t + l16];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[i][nt] = mfma16x16x4(a, pfull[nt * 272 + (4 * g + s) * 17 + l16], acc[i][nt]);
        }
      }
    }
  }
  // epilogue: this workgroup's partial (rows = concatenated columns of A)
  const int W_out = NB * k;
  CT* out = partial + (int64_t)rg * D * W_out;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int t = tbeg + w + kPassWaves * i;
    if (t < tend) {
      const bool b1 = (NB == 2) && (t >= T0);
      const int db = b1 ? d1 : d0;
      const int ct = b1 ? t - T0 : t;
      const int rowbase = b1 ? d0 : 0;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int bsrc = nt / KT, kt = nt % KT;
        const int col = kt * 16 + l16;
        if (col < k) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int c = ct * 16 + acc_row<CT>(lane, r);
            if (c < db) out[(int64_t)(rowbase + c) * W_out + bsrc * k + col] = acc[i][nt][r];
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------
// FP32 data and arithmetic: the same products with the row blocks moved
// straight from HBM into LDS by the load unit (buffer loads with the LDS
// flag, no VGPRs), double-buffered, so a workgroup can own whole rows:
//   * 8-row blocks; block i+1 streams into the second LDS buffer while the
//     matrix cores work on block i, and the only wait on it is at the top
//     of the next iteration;
//   * the barriers inside an iteration wait on LDS traffic only (an LDS
//     fence would also wait on the in-flight block);
//   * the direction operands of a wave's tiles stay in registers for the
//     launch, and each wave accumulates A_b^T [P_0 | P_1] for the same
//     tiles it used for P (no column split, no duplicated P).
// Tile t of [A_0 | A_1] (16 columns; A_1's tiles follow A_0's) sits at LDS
// column 16 t, so every operand address is one base register plus a
// compile-time offset.  A load instruction moves CH = 64 VEC consecutive
// floats of one row; the last chunk of each block is shifted back to end
// on the block's last tile (it rewrites identical values), so no chunk
// spills into the other block's columns.  The row pitch is 4 mod 32 floats
// (bank-conflict free for both operand patterns).  The 16 MFMA rows of the
// P products hold the block's 8 rows twice: rows 0-7 accumulate A_0 W_0 and
// rows 8-15 A_1 W_1 (each lane zeroes the operand of the other view), so
// one accumulator serves both views and the tile loop has no view branch.
constexpr int kDmaRows = 8;
constexpr int kDmaMaxTiles = 128;   // 2048 columns of [A_0 | A_1]
// The FP32 pass runs 16 waves (4 per SIMD, 128 registers each): a wave
// holds the direction operands and the J accumulators of at most 8 tiles.
constexpr int kF32Waves = 16;
constexpr int kF32Threads = 64 * kF32Waves;

__device__ __forceinline__ void lds_only_barrier() {
  // LDS traffic of this wave done, then the workgroup barrier; in-flight
  // global-to-LDS loads of the next block are deliberately not waited on.
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// NT: the non-temporal hint (data that no cache keeps until its next use).
template <int VEC, bool NT = false>
__device__ __forceinline__ void dma_row_chunk(__amdgpu_buffer_rsrc_t r, float* lds_dst, int voff) {
  if constexpr (VEC == 4 && NT)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds_dst, 16, voff, 0, 0, 2);
  else if constexpr (VEC == 4)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds_dst, 16, voff, 0, 0, 0);
  else
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds_dst, 4, voff, 0, 0, 0);
}

__host__ __device__ constexpr int dma_pitch(int TT) { return ((TT * 16 + 31) / 32) * 32 + 4; }

template <int TPB, int VEC>
__global__ void __launch_bounds__(kF32Threads) k_pass_dma(const float* __restrict__ A0, const float* __restrict__ A1,
                                                          int64_t n, int d0, int d1, int k,
                                                          const float* __restrict__ Wp0,
                                                          const float* __restrict__ Wp1, int nrb,
                                                          float* __restrict__ partial, const int* __restrict__ done) {
  if (done && *done) return;
  constexpr int R = kDmaRows;
  constexpr int CH = 64 * VEC;
  constexpr int NT = 2;                                         // [P_0 | P_1] tiles of the J phase
  using acc_t = f32x4;
  extern __shared__ float dsm[];
  const int T0 = (d0 + 15) >> 4;
  const int T1 = (d1 + 15) >> 4;
  const int TT = T0 + T1;
  const int nch0 = (T0 * 16 + CH - 1) / CH, nch1 = (T1 * 16 + CH - 1) / CH;
  const int nch = nch0 + nch1;
  const int pitch = dma_pitch(kF32Waves * TPB);
  float* red = dsm + 2 * R * pitch;              // [waves][16 x 16]
  float* pfull = red + kF32Waves * 256;          // [2][R][17]

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const __amdgpu_buffer_rsrc_t wr0 = make_rsrc(Wp0, (int64_t)T0 * 16 * 16 * 4);
  const __amdgpu_buffer_rsrc_t wr1 = make_rsrc(Wp1, (int64_t)T1 * 16 * 16 * 4);
  const int wvoff = (g * 16 + l16) * 4;

  // Slot i of wave w is tile t = w + 16 i (TPB >= the tiles / 16); slots past
  // the last tile have a zero direction operand and read zero LDS columns,
  // so every wave runs the same branch-free instruction stream.  keep[i]
  // zeroes, in the P products, the lanes of MFMA rows that belong to the
  // other view (rows 0-7: A_0, rows 8-15: A_1).
  float wreg[TPB][4];
  uint32_t keep[TPB];
  acc_t acc[TPB][NT];
#pragma unroll
  for (int i = 0; i < TPB; ++i) {
    const int t = w + kF32Waves * i;
    const bool b1 = t >= T0;
    keep[i] = (l16 >> 3) == (int)b1 ? ~0u : 0u;
    const int ct = b1 ? t - T0 : t;
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      const int soff = (ct * 16 + 4 * s2) * 16 * 4;
      float v = 0.f;
      if (t < TT) v = b1 ? buf_load<float>(wr1, wvoff + soff, 0) : buf_load<float>(wr0, wvoff + soff, 0);
      wreg[i][s2] = v;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
  }
  // The columns of the slots past the last tile are never loaded: zero both
  // row buffers once.
  for (int e = tid; e < 2 * R * pitch; e += kF32Threads) dsm[e] = 0.f;
  __syncthreads();

  // Loads of row block rbk into buffer xb: wave w moves chunks j = w, w + 16,
  // ... of every row.  One buffer resource per view and block; rows past n
  // lie past its num_records and read as zero.  A chunk's tail past the
  // view's last column reads the next row's leading values, which
  // clear_block takes out.
  auto issue_block = [&](int rbk, float* xb) __attribute__((always_inline)) {
    const int64_t row0 = (int64_t)rbk * R;
    const int rows = (int)(n - row0 < R ? n - row0 : R);
    const __amdgpu_buffer_rsrc_t r0 = make_rsrc(A0 + row0 * d0, (int64_t)rows * d0 * 4);
    const __amdgpu_buffer_rsrc_t r1 = make_rsrc(A1 + row0 * d1, (int64_t)rows * d1 * 4);
    for (int j = w; j < nch; j += kF32Waves) {
      const bool s1 = j >= nch0;
      const int jj = s1 ? j - nch0 : j;
      const int span = (s1 ? T1 : T0) * 16;
      const int o = min(jj * CH, span - CH);
      const int db4 = (s1 ? d1 : d0) * 4;
      float* dst = xb + (s1 ? T0 * 16 : 0) + o;
      const int vbase = (o + lane * VEC) * 4;
      const __amdgpu_buffer_rsrc_t rs = s1 ? r1 : r0;
#pragma unroll
      for (int r = 0; r < R; ++r) dma_row_chunk<VEC>(rs, dst + r * pitch, vbase + r * db4);
    }
  };

  // The columns between a view's last and its last tile's, zeroed by the wave
  // that loaded them: they meet zero direction rows in P, but an infinity or a
  // NaN of the next row would turn this row's P into NaN.
  auto clear_block = [&](float* xb) __attribute__((always_inline)) {
    static_assert(R == 8, "four rows a store, two stores");
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int c = (v ? d1 : d0) + l16, span = (v ? T1 : T0) * 16;
      if (w == ((v ? nch : nch0) - 1) % kF32Waves && c < span) {
        float* x = xb + g * pitch + (v ? T0 * 16 : 0) + c;
        x[0] = 0.f;
        x[4 * pitch] = 0.f;
      }
    }
  };

  // per-lane operand bases (floats); slot i adds 16 (w + 16 i)
  const int base_b = (l16 & (R - 1)) * pitch + g + 16 * w;   // P phase: row l16 mod 8, column 4 s2 + g
  const int base_d = g * pitch + l16 + 16 * w;               // J phase: row g + 4 s, column l16
  const int pf_b = g * 17 + l16;                              // pfull row g + 4 s (as the J-phase A operand)

  int rb = blockIdx.x;
  int boff = 0;   // float offset of the current buffer
  if (rb < nrb) issue_block(rb, dsm);
  for (; rb < nrb; rb += gridDim.x) {
    __builtin_amdgcn_s_waitcnt(0);   // this wave's loads of the block have landed
    clear_block(dsm + boff);
    __syncthreads();                 // ... and every wave's; the other buffer is free
    const float* xs = dsm + boff;
    if (rb + (int)gridDim.x < nrb) issue_block(rb + gridDim.x, dsm + (R * pitch - boff));
    // (b) P partials over this wave's slots.  Both views share one
    // accumulator: MFMA rows 0-7 take A_0 W_0 (the lanes of rows 8-15 read
    // zero on A_0 tiles) and rows 8-15 take A_1 W_1; two accumulators
    // alternate to break the dependence chain.
    acc_t pacc[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
    for (int i = 0; i < TPB; ++i) {
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        const float a = __builtin_bit_cast(
            float, __builtin_bit_cast(uint32_t, xs[base_b + 16 * kF32Waves * i + 4 * s2]) & keep[i]);
        pacc[i & 1] = mfma16x16x4(a, wreg[i][s2], pacc[i & 1]);
      }
    }
    // (c) sum P over the waves
#pragma unroll
    for (int r = 0; r < 4; ++r) red[w * 256 + (4 * g + r) * 16 + l16] = pacc[0][r] + pacc[1][r];
    lds_only_barrier();
    if (tid < 2 * R * 16) {
      float v = 0.f;
#pragma unroll
      for (int ww = 0; ww < kF32Waves; ++ww) v += red[ww * 256 + tid];
      const int row = tid >> 4, col = tid & 15;
      pfull[(row >> 3) * (R * 17) + (row & 7) * 17 + col] = v;
    }
    lds_only_barrier();
    // (d) A_b^T [P_0 | P_1] for this wave's slots
    float pb[R / 4][NT];
#pragma unroll
    for (int s = 0; s < R / 4; ++s)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) pb[s][nt] = pfull[nt * (R * 17) + pf_b + 4 * s * 17];
#pragma unroll
    for (int i = 0; i < TPB; ++i) {
#pragma unroll
      for (int s = 0; s < R / 4; ++s) {
        const float a = xs[base_d + 4 * s * pitch + 16 * kF32Waves * i];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[i][nt] = mfma16x16x4(a, pb[s][nt], acc[i][nt]);
      }
    }
    boff = R * pitch - boff;
  }
  // epilogue: this workgroup's partial (rows = concatenated columns of A)
  const int W_out = 2 * k;
  const int D = d0 + d1;
  float* out = partial + (int64_t)blockIdx.x * D * W_out;
#pragma unroll
  for (int i = 0; i < TPB; ++i) {
    const int t = w + kF32Waves * i;
    if (t < TT) {
      const bool b1 = t >= T0;
      const int db = b1 ? d1 : d0;
      const int ct = b1 ? t - T0 : t;
      const int rowbase = b1 ? d0 : 0;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int col = l16;
        if (col < k) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int c = ct * 16 + acc_row<float>(lane, r);
            if (c < db) out[(int64_t)(rowbase + c) * W_out + nt * k + col] = acc[i][nt][r];
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------
// FP32, one or two views: the narrow products on 4x4 matrix-core blocks
// (v_mfma_f32_4x4x1f32: sixteen independent 4 x 4 outer products per
// instruction; 16 x 16 tiles would carry mostly zero padding for a few rows
// and k columns), the two products of a block of R rows pipelined over two
// sets of waves:
//   * the loader wave moves the rows HBM -> LDS (buffer loads with the LDS
//     flag) into a ring of four blocks.  A wave that issues loads stalls
//     while the load queue is full, so none of the others does.
//   * eight producer waves form P_b = A_b W_b: half of them take a view (all
//     with one view) and own groups of four of its tiles; an instruction
//     takes a group, 4 rows x 4 direction columns per tile over one of every
//     four of its columns.  The four tiles are summed in registers by
//     lane-row swaps and the column phases by two DPP rotations: one partial
//     per wave, into LDS.
//   * seven consumer waves add the producers' partials in wave order as they
//     read them and accumulate J_b = A_b^T [P_0 | P_1] over runs of
//     neighbouring tiles: whole 16-column tiles of [P_0 | P_1] on 16x16x4
//     products, the remaining 4-column groups on 4x4 blocks, one row of the
//     block per instruction over four tiles at once (the 16-lane rows take
//     the tiles, the blocks of a row 4 of its columns).  [P_0 | P_1] is
//     packed tight (C4 groups of 4).
// In step i the loader issues block i + 2 and waits for block i + 1 (issued
// a step earlier), the producers multiply block i and the consumers work on
// block i - 1; one barrier per step.  R rows a block, by the width, so that
// a step is 33 KB of LDS for every width and its fixed cost is spread alike.
//
// Bounds: the row stream up to about 8 direction columns of [P_0 | P_1]
// (6.7 TB/s), past that the products: the producers' chain (LDS reads,
// products, lane sums, partials) and the consumers' on the same SIMDs.
// Measured, us, against one set of 16 waves that did both products in turn
// (two barriers more a block, and 4-byte loads for odd widths):
//   200000 x (1000 + 1000), k = 10   377 -> 335 (4.8 TB/s)   k = 3  250 -> 240
//   100000 x 2000, k = 19            236 -> 220              k = 9  159 -> 143
//   52345 x (531 + 347), k = 9       99 -> 59                20011 x (301 + 203), k = 8  24 -> 20
//   100000 x (250 + 256), k = 10     121 -> 68               200000 x (64 + 50), k = 4   132 -> 58
template <int N>
__device__ __forceinline__ float dpp_row_ror(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + N, 0xF, 0xF, false));
}
__device__ __forceinline__ f32x4 mfma4x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// Sums of the four values x[0..3] over the four 16-lane rows, scattered:
// afterwards 16-lane row g holds the sum of x[r], r = (0, 2, 1, 3)[g].
// v_permlane32_swap exchanges the upper half of its first operand with the
// lower half of its second, so the sum of the swapped pair (x[0], x[1])
// holds x[0] over rows (g, g + 2) in rows 0-1 and x[1] in rows 2-3;
// v_permlane16_swap (odd rows of the first operand with even rows of the
// second) then finishes two such pairs in one step.  Four swaps and four
// adds reduce four values, against two swaps and three adds per value for
// separate full sums.
__device__ __forceinline__ float rows_scatter_sum(f32x4 x) {
  auto u = [](float v) { return __builtin_bit_cast(uint32_t, v); };
  auto f = [](uint32_t v) { return __builtin_bit_cast(float, v); };
  const auto a = __builtin_amdgcn_permlane32_swap(u(x[0]), u(x[1]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(u(x[2]), u(x[3]), false, false);
  const float p = f(a[0]) + f(a[1]), q = f(b[0]) + f(b[1]);
  const auto c = __builtin_amdgcn_permlane16_swap(u(p), u(q), false, false);
  return f(c[0]) + f(c[1]);
}

constexpr int kPipeProd = 8;    // producer waves: 0 .. 7
constexpr int kPipeCons = 7;    // consumer waves: 8 .. 14; wave 15 loads
constexpr int kPipeRing = 4;    // blocks of rows in LDS

// R rows a block (4, 8 or 16 for up to 128, 64 or 32 tiles of [A_0 | A_1]);
// C4 4-column groups of [P_0 | P_1]; PG_ 4-tile groups a producer may hold.
template <int NV, int R_, int C4, int PG_>
struct PipeShape {
  static constexpr int R = R_;
  static constexpr int TILES = 512 / R;            // most tiles
  static constexpr int SLOTS = (TILES + kPipeCons - 1) / kPipeCons;   // tiles of a consumer
  static constexpr int NG = (SLOTS + 3) / 4;       // 4-tile groups of a consumer
  static constexpr int KG = NV == 2 ? (C4 + 1) / 2 : C4;   // 4-column groups of one view's P
  static constexpr int JQ = (C4 + 2) / 4;          // 16-column tiles of [P_0 | P_1]
  static constexpr int JR = C4 % 4 == 1 ? 1 : 0;   // a single 4-column group past them (two or three: a tile)
  static constexpr int PG = PG_;
  static constexpr int NPV = kPipeProd / NV;       // producers of a view
  // one view: a producer's groups that are whole in every wave (an instance
  // of PG groups serves widths that need more than PG / 2 of them)
  static constexpr int FULL = NV == 1 ? PG / 2 : 0;
  // a producer's sums for 8 rows and KH direction-column groups at a time,
  // its operands for BT tile groups at a time: beside its directions they
  // take at most 96 of a wave's 128 registers.  One group at a time is read
  // ahead of its use instead (AHEAD): 2000 columns, k = 19: 245 us without
  static constexpr int RB = R < 8 ? R : 8;
  static constexpr bool over(int kh, int b) { return 4 * KG * PG + RB * kh + b * RB > 96; }
  static constexpr int KH = over(KG, 1) ? (KG + 1) / 2 : KG;
  static constexpr int bt(int b) { return b > 1 && (b > PG || over(KH, b)) ? bt(b / 2) : b; }
  static constexpr int BT = bt(4);
  static constexpr bool AHEAD = BT == 1 && PG > 1;
  // row pitch in floats, 16 mod 64: four rows of 16 consecutive columns (a
  // consumer's operand) fall on 64 distinct banks, as do the producers'
  // column quadruples of one 16-lane row
  static constexpr int PITCH = 16 * TILES + 16;
  static constexpr int BUF = R * PITCH;
  // the partials of one element of P lie side by side (8 floats: a
  // consumer reads its view's four, or all eight, in 16-byte loads)
  static constexpr int PART = R * 4 * KG * kPipeProd;
  static constexpr size_t lds_bytes() { return (size_t)(kPipeRing * BUF + 2 * PART) * 4; }
};

// The loader's loads of the R rows at a0 (and a1), `left` of them before the
// end of the data, into dst: chunks of 256 columns (16 bytes a lane), rows
// past the end read zero through the resource's range check.  Columns
// between a view's last and its last tile's read the next row's first
// values (they stay out of P and land in J rows that are not stored).  Rows
// need not start on 16-byte boundaries (a 16-byte load takes any 4-byte one);
// but a load that straddles the end of the matrix must not lose its valid part
// to the range check, so the block with the last row is loaded 4 bytes a lane
// when a row is no multiple of 16 bytes.  Returns the number of loads in
// flight for the block (0 stands for "wait for all").
template <int NV, int R, int PITCH, bool NT>
__device__ __forceinline__ int pipe_load(const float* a0, const float* a1, int64_t left, int d0, int d1, int T0,
                                         int T1, float* __restrict__ dst, int lane) {
  const bool tail = left <= R && ((d0 | d1) & 3) != 0;
  int cnt = 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int dv = v ? d1 : d0, span = (v ? T1 : T0) * 16;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(v ? a1 : a0, left * dv * 4);
    float* dv0 = dst + (v ? T0 * 16 : 0);
    if (!tail) {
      // whole chunks, then the part of one that is left
      int c0 = 0;
      for (; c0 + 256 <= span; c0 += 256)
#pragma unroll
        for (int r = 0; r < R; ++r) dma_row_chunk<4, NT>(rs, dv0 + r * PITCH + c0, (r * dv + c0 + 4 * lane) * 4);
      if (c0 + 4 * lane < span)
#pragma unroll
        for (int r = 0; r < R; ++r) dma_row_chunk<4, NT>(rs, dv0 + r * PITCH + c0, (r * dv + c0 + 4 * lane) * 4);
      cnt += R * ((span + 255) / 256);
    } else {
      for (int c0 = 0; c0 < span; c0 += 64)
        if (c0 + lane < span)
#pragma unroll
          for (int r = 0; r < R; ++r) dma_row_chunk<1>(rs, dv0 + r * PITCH + c0, (r * dv + c0 + lane) * 4);
    }
  }
  return tail ? 0 : cnt;
}

// At most n of this wave's loads outstanding (n a multiple of 4: blocks are
// 4, 8 or 16 loads a chunk of columns; gfx9 encoding of vmcnt).
__device__ __forceinline__ void pipe_wait(int n) {
  switch (n) {
#define SRP_VM(N) case N: __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8)); break;
    SRP_VM(4) SRP_VM(8) SRP_VM(12) SRP_VM(16) SRP_VM(20) SRP_VM(24) SRP_VM(28) SRP_VM(32) SRP_VM(36) SRP_VM(40)
    SRP_VM(48)
#undef SRP_VM
    default: __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));
  }
}

// Zeroes the columns c .. end - 1 (at most three) of the block in xs that
// share a quadruple of columns with a view's last: they meet zero direction
// rows in P, but an infinity or a NaN of the next row there would turn this
// row's P into NaN.  The wave that owns the tile does it before its own reads,
// which follow in order (the loader, after its wait for the block: 200000 x
// (66 + 50), k = 4 83 -> 88 us a call, here 83).
template <class S>
__device__ __forceinline__ void pipe_clear(float* xs, int c, int end, int lane) {
  asm volatile("");   // keeps the caller's test a scalar branch, which the other waves take
  c += lane & 3;
  if (c < end && lane < 4 * S::R) xs[(lane >> 2) * S::PITCH + c] = 0.f;
}

// A producer's partial of P for the block in xs (ngrp groups).  pcol: the
// LDS column of this lane's quadruple in group 0; nok: groups whose quadruple
// of this lane exists (the zeros of the row's padding stand for the rest).
template <class S>
__device__ __forceinline__ void pipe_produce(const float* __restrict__ xs, float* __restrict__ part, int w, int lane,
                                             int ngrp, const float (&wreg)[S::PG][4][S::KG], int pcol, int nok) {
  constexpr int R = S::R, KG = S::KG, PG = S::PG, RG = S::RB / 4, KH = S::KH, BT = S::BT;
  // lane-dependent offsets are formed per block: live across the loop they
  // would spill beside the directions
  asm volatile("" : "+v"(lane), "+v"(pcol), "+v"(nok));
  const int g = lane >> 4, cs = (lane >> 2) & 3, q4 = lane & 3;
  const float* xq = xs + q4 * S::PITCH;
  // items: batches of BT groups, in turn for each half of the directions and
  // each RB rows
  constexpr int NBT = (PG + BT - 1) / BT, NK = (KG + KH - 1) / KH, NIT = R / S::RB * NK * NBT;
  float4 a4[S::AHEAD ? 2 : 1][BT][RG];
  auto read = [&](int it) __attribute__((always_inline)) {
    const int b = it % NBT * BT, r0 = it / (NBT * NK) * S::RB;
#pragma unroll
    for (int u = 0; u < BT; ++u)
#pragma unroll
      for (int rg = 0; rg < RG; ++rg)
        a4[S::AHEAD ? it & 1 : 0][u][rg] = *reinterpret_cast<const float4*>(
            xq + (r0 + 4 * rg) * S::PITCH +
            (b + u < S::FULL || b + u < nok ? pcol + 64 * S::NPV * (b + u) : S::PITCH - 16));
  };
  f32x4 pacc[RG][KH];
  if (S::AHEAD) read(0);
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int b = it % NBT * BT, k0 = it / NBT % NK * KH, r0 = it / (NBT * NK) * S::RB;
    if (b == 0)
#pragma unroll
      for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int kk = 0; kk < KH; ++kk) pacc[rg][kk] = f32x4{0, 0, 0, 0};
    if (S::AHEAD) {
      if (it + 1 < NIT) read(it + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (b < S::FULL || b < ngrp) {
      if (!S::AHEAD) read(it);
#pragma unroll
      for (int u = 0; u < BT; ++u)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int rg = 0; rg < RG; ++rg) {
            const float4 a = a4[S::AHEAD ? it & 1 : 0][u][rg];
            const float av = s == 0 ? a.x : s == 1 ? a.y : s == 2 ? a.z : a.w;
#pragma unroll
            for (int kk = 0; kk < KH; ++kk)
              if (k0 + kk < KG) pacc[rg][kk] = mfma4x4(av, wreg[b + u][s][k0 + kk], pacc[rg][kk]);
          }
    }
    if (b + BT >= PG) {
      // the four tiles of a 16-lane row by a scattered row sum, then the
      // column phases: lane (g, 0, q4) holds row r0 + 4 rg + (0, 2, 1, 3)[g],
      // direction column 4 (k0 + kk) + q4
      const int r = ((g & 1) << 1) | (g >> 1);
      float* rw = part + ((r0 + r) * (4 * KG) + 4 * k0 + q4) * kPipeProd + w;
#pragma unroll
      for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int kk = 0; kk < KH; ++kk)
          if (k0 + kk < KG) {
            float x = rows_scatter_sum(pacc[rg][kk]);
            x += dpp_row_ror<4>(x);
            x += dpp_row_ror<8>(x);
            asm volatile("" : "+v"(x));   // the sum in every lane: both rotations fold into the adds
            if (cs == 0) rw[(rg * 16 * KG + 4 * kk) * kPipeProd] = x;
          }
    }
  }
}

// An element of [P_0 | P_1]: its view's partials in wave order.
template <int NV>
__device__ __forceinline__ float pipe_sum(const float* p) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  float s = ((a.x + a.y) + a.z) + a.w;
  if constexpr (NV == 1) {
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    s = (((s + b.x) + b.y) + b.z) + b.w;
  }
  return s;
}

// A consumer's step: J += A_b^T [P_0 | P_1] over this wave's first 4 NACT
// tiles (its groups that hold any), P from the producers' partials.  xs: the
// block at this wave's first tile.  pq, pr: this lane's element of a row of
// P for column l16 of the whole tiles and column q4 of the groups past them.
// The order of reads and products is the compiler's: reads two batches ahead
// behind scheduling barriers come in bursts that hold up the loader's writes
// (200000 x (1000 + 1000), k = 10: 364 us, 335 so).
template <class S, int NV, int NACT>
__device__ __forceinline__ void pipe_consume(const float* __restrict__ xs, const float* __restrict__ part, int lane,
                                             const int (&pq)[2], const int (&pr)[3],
                                             f32x4 (&acc)[S::SLOTS][S::JQ > 0 ? S::JQ : 1],
                                             f32x4 (&accr)[S::NG][S::JR > 0 ? S::JR : 1]) {
  constexpr int R = S::R, KG = S::KG, JQ = S::JQ, JR = S::JR;
  constexpr int NS = 4 * NACT < S::SLOTS ? 4 * NACT : S::SLOTS;   // tiles
  constexpr int ROW = 4 * KG * kPipeProd;   // floats per row of the partials
  const int g = lane >> 4, l16 = lane & 15;
#pragma unroll
  for (int h = 0; h < R / 4; ++h) {   // four rows at a time
    // whole tiles: lane row g takes block row 4 h + g, a tile per product;
    // 4x4 blocks: a row per product, lane row g takes its tile 4 G + g
    const float* xq = xs + (4 * h + g) * S::PITCH + l16;
    const float* xr = xs + 4 * h * S::PITCH + lane;
    float pbq[JQ > 0 ? JQ : 1], pbr[4][JR > 0 ? JR : 1];
#pragma unroll
    for (int jq = 0; jq < JQ; ++jq) pbq[jq] = pipe_sum<NV>(part + (4 * h + g) * ROW + pq[jq]);
#pragma unroll
    for (int jr = 0; jr < JR; ++jr) {
      // this lane row's element; swaps then give every lane row each of the
      // four: the swap of a value with its copy leaves lane rows 0 1 0 1 in
      // one and 2 3 2 3 in the other, the next ones a row each.
      const uint32_t x = __builtin_bit_cast(uint32_t, pipe_sum<NV>(part + (4 * h + g) * ROW + pr[jr]));
      const auto y = __builtin_amdgcn_permlane32_swap(x, x, false, false);
      const auto z0 = __builtin_amdgcn_permlane16_swap(y[0], y[0], false, false);
      const auto z1 = __builtin_amdgcn_permlane16_swap(y[1], y[1], false, false);
      const uint32_t z[4] = {z0[0], z0[1], z1[0], z1[1]};
#pragma unroll
      for (int rho = 0; rho < 4; ++rho) pbr[rho][jr] = __builtin_bit_cast(float, z[rho]);
    }
    if constexpr (JQ > 0)
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const float a = xq[16 * t];
#pragma unroll
        for (int jq = 0; jq < JQ; ++jq) acc[t][jq] = mfma16x16x4(a, pbq[jq], acc[t][jq]);
      }
    if constexpr (JR > 0)
#pragma unroll
      for (int rho = 0; rho < 4; ++rho)
#pragma unroll
        for (int G = 0; G < NACT; ++G) {
          const float a = xr[rho * S::PITCH + 64 * G];
#pragma unroll
          for (int jr = 0; jr < JR; ++jr) accr[G][jr] = mfma4x4(a, pbr[rho][jr], accr[G][jr]);
        }
  }
}

template <int NV, int R_, int C4, int PG_>
__global__ void __launch_bounds__(kF32Threads) k_pass_quad(const float* __restrict__ A0, const float* __restrict__ A1,
                                                           int64_t n, int d0, int d1, int k,
                                                           const double* __restrict__ W0,
                                                           const double* __restrict__ W1, int nrb,
                                                           float* __restrict__ partial, const int* __restrict__ done) {
  if (done && *done) return;
  using S = PipeShape<NV, R_, C4, PG_>;
  constexpr int R = S::R, KG = S::KG, JQ = S::JQ, JR = S::JR, NG = S::NG, PG = S::PG;
  extern __shared__ float dsm[];
  float* parts = dsm + kPipeRing * S::BUF;   // two sets of partials
  const int T0 = (d0 + 15) >> 4, T1 = NV == 2 ? (d1 + 15) >> 4 : 0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this workgroup's blocks: pairs of neighbours, pair blockIdx.x + j grid
  // (twice the run of bytes: the row stream alone takes 264 us against 279
  // with single blocks, 200000 x (1000 + 1000))
  const int pairs = (nrb + 1) / 2, mine = (pairs - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  const int nst = 2 * mine - ((nrb & 1) && (pairs - 1) % (int)gridDim.x == (int)blockIdx.x ? 1 : 0);
  if (w == kPipeProd + kPipeCons) {
    auto stream = [&](auto nt_) __attribute__((always_inline)) {
      int64_t row = (int64_t)blockIdx.x * 2 * R;
      auto load = [&](int i) __attribute__((always_inline)) {   // block i, at `row`
        const int cnt = pipe_load<NV, R, S::PITCH, decltype(nt_)::value>(
            A0 + row * d0, NV == 2 ? A1 + row * d1 : nullptr, n - row, d0, NV == 2 ? d1 : 0, T0, T1,
            dsm + (i & 3) * S::BUF, lane);
        row += (i & 1) ? (2ll * gridDim.x - 1) * R : R;
        return cnt;
      };
      load(0);
      pipe_wait(nst > 1 ? load(1) : 0);   // block 0 has landed
      lds_only_barrier();
      for (int i = 0; i <= nst; ++i) {
        pipe_wait(i + 2 < nst ? load(i + 2) : 0);   // block i + 1 has landed; block i + 2 stays in flight
        lds_only_barrier();
      }
    };
    // data past the 256 MB that the memory-side cache holds is read once per
    // pass: without the hint its stream runs at 5.9 TB/s, with it at 6.7
    // (100000 x (1000 + 1000), k = 1: 135 and 120 us); data that fits is
    // still there in the next pass (3000 x 2000, k = 9: 19 us, with the hint 22)
    if (n * (d0 + (NV == 2 ? d1 : 0)) * 4 > (256ll << 20)) stream(std::integral_constant<bool, true>{});
    else stream(std::integral_constant<bool, false>{});
  } else if (w < kPipeProd) {
    const int g = lane >> 4, cs = (lane >> 2) & 3, q4 = lane & 3;
    // this wave's direction operands: group G is tiles 4 (wl + NPV G) .. + 3
    // of its view, lane (g, cs, q4) holds direction column 4 kg + q4 for
    // column 4 cs + s of tile g, read from the FP64 directions (rows past d
    // lie past the resource and read zero, columns past k and tiles past the
    // last take the zero offset)
    const bool v1 = w >= S::NPV;   // NV == 1: never
    const int wl = v1 ? w - S::NPV : w;
    const int Tv = v1 ? T1 : T0;
    const int ngrp = (((Tv + 3) >> 2) - wl + S::NPV - 1) / S::NPV;
    const int dv = v1 ? d1 : d0;
    const __amdgpu_buffer_rsrc_t wrs = make_rsrc(v1 ? W1 : W0, (int64_t)dv * k * 8);
    float wreg[PG][4][KG];
    const int pcol = 16 * ((v1 ? T0 : 0) + 4 * wl + g) + 4 * cs;
    const int tend = 16 * (Tv - 1) + 4 * cs < dv ? Tv : Tv - 1;   // tiles with this lane's quadruple
    const int nok = (tend - (4 * wl + g) + 4 * S::NPV - 1) / (4 * S::NPV);   // <= 0 where the first is past the last
    // the wave with the view's last tile clears what its last quadruple has past the view
    const int clast = (v1 ? 16 * T0 : 0) + dv, cend = (clast + 3) & ~3;
    const bool clears = clast < cend && ((Tv - 1) >> 2) % S::NPV == wl;
    // the padding of the ring's rows, which no load touches
    for (int e = tid; e < kPipeRing * R * 16; e += 64 * kPipeProd) dsm[(e >> 4) * S::PITCH + S::PITCH - 16 + (e & 15)] = 0.f;
#pragma unroll
    for (int G = 0; G < PG; ++G) {
      const int tv = 4 * (wl + S::NPV * G) + g;
      const bool ok = tv < Tv;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int kg = 0; kg < KG; ++kg) {
          const int col = 4 * kg + q4;
          const int off = (ok && col < k) ? ((16 * tv + 4 * cs + s) * k + col) * 8 : kOob;
          wreg[G][s][kg] = (float)buf_load<double>(wrs, off, 0);
        }
    }
    lds_only_barrier();
    for (int i = 0; i <= nst; ++i) {
      if (i < nst) {
        if (clears) pipe_clear<S>(dsm + (i & 3) * S::BUF, clast, cend, lane);
        pipe_produce<S>(dsm + (i & 3) * S::BUF, parts + (i & 1) * S::PART, w, lane, ngrp, wreg, pcol, nok);
      }
      lds_only_barrier();
    }
  } else {
    const int wj = w - kPipeProd;
    const int g = lane >> 4, l16 = lane & 15, cs = (lane >> 2) & 3, q4 = lane & 3;
    const int TT = T0 + T1;
    const int per = (TT + kPipeCons - 1) / kPipeCons;   // tiles of a consumer: per wj .. per wj + per - 1
    f32x4 acc[S::SLOTS][JQ > 0 ? JQ : 1];
    f32x4 accr[NG][JR > 0 ? JR : 1];
#pragma unroll
    for (int i = 0; i < S::SLOTS; ++i)
#pragma unroll
      for (int j = 0; j < (JQ > 0 ? JQ : 1); ++j) acc[i][j] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int G = 0; G < NG; ++G)
#pragma unroll
      for (int j = 0; j < (JR > 0 ? JR : 1); ++j) accr[G][j] = f32x4{0, 0, 0, 0};
    // column c of [P_0 | P_1] is column c - v k of view v (columns past the
    // last read the last's; their sums are not stored)
    const int cmax = NV * k - 1;
    int pq[2] = {0, 0}, pr[3] = {0, 0, 0};
    auto element = [&](int c) {
      c = min(c, cmax);
      const int v = c >= k ? 1 : 0;
      return (c - v * k) * kPipeProd + v * S::NPV;
    };
#pragma unroll
    for (int jq = 0; jq < JQ; ++jq) pq[jq] = element(16 * jq + l16);
#pragma unroll
    for (int jr = 0; jr < JR; ++jr) pr[jr] = element(16 * JQ + 4 * jr + q4);
    lds_only_barrier();
    lds_only_barrier();   // the producers' step 0
    auto steps = [&](auto n_) __attribute__((always_inline)) {
      for (int i = 0; i < nst; ++i) {
        pipe_consume<S, NV, decltype(n_)::value>(dsm + (i & 3) * S::BUF + 16 * per * wj, parts + (i & 1) * S::PART,
                                                 lane, pq, pr, acc, accr);
        lds_only_barrier();
      }
    };
    const int nact = (per + 3) / 4;
    if (NG == 1 || nact == 1) steps(std::integral_constant<int, 1>{});
    else if (NG == 2 || nact == 2) steps(std::integral_constant<int, 2>{});
    else if (NG == 3 || nact == 3) steps(std::integral_constant<int, NG < 3 ? 1 : 3>{});
    else if (nact == 4) steps(std::integral_constant<int, NG < 4 ? 1 : 4>{});
    else steps(std::integral_constant<int, NG < 5 ? 1 : 5>{});
    // this workgroup's partial (rows = concatenated columns of A, columns =
    // [P_0 | P_1])
    const int W_out = NV * k;
    float* out = partial + (int64_t)blockIdx.x * (d0 + (NV == 2 ? d1 : 0)) * W_out;
    auto put = [&](int slot, int row, int c, float x) __attribute__((always_inline)) {
      const int t = per * wj + slot;
      const bool b1 = NV == 2 && t >= T0;
      const int rv = 16 * (b1 ? t - T0 : t) + row;
      if (slot < per && t < TT && c < W_out && rv < (b1 ? d1 : d0)) out[(int64_t)((b1 ? d0 : 0) + rv) * W_out + c] = x;
    };
    if constexpr (JQ > 0) {
#pragma unroll
      for (int i = 0; i < S::SLOTS; ++i)
#pragma unroll
        for (int jq = 0; jq < JQ; ++jq)
#pragma unroll
          for (int r = 0; r < 4; ++r) put(i, acc_row<float>(lane, r), 16 * jq + l16, acc[i][jq][r]);
    }
    if constexpr (JR > 0) {
#pragma unroll
      for (int G = 0; G < NG; ++G)
#pragma unroll
        for (int jr = 0; jr < JR; ++jr)
#pragma unroll
          for (int r = 0; r < 4; ++r) put(4 * G + g, 4 * cs + r, 16 * JQ + 4 * jr + q4, accr[G][jr][r]);
    }
  }
}

// Tile slots per wave: the smaller instance covering the tiles of
// [A_0 | A_1] (two views of at most 64 tiles together take k_pass_quad).
static int dma_slots(int d0, int d1) {
  const int TT = (d0 + 15) / 16 + (d1 + 15) / 16;
  return TT <= 6 * kF32Waves ? 6 : 8;
}

static size_t dma_lds_bytes(int d0, int d1) {
  const size_t pitch = (size_t)dma_pitch(kF32Waves * dma_slots(d0, d1));
  return (2 * kDmaRows * pitch + (size_t)kF32Waves * 256 + (size_t)2 * kDmaRows * 17) * sizeof(float);
}

// 16-byte loads need rows that start on 16-byte boundaries and blocks of
// at least 16 tiles (one 256-float chunk); 4-byte loads blocks of 4 tiles.
static int dma_vec(const void* A0, const void* A1, int d0, int d1) {
  const int T0 = (d0 + 15) / 16, T1 = (d1 + 15) / 16;
  const bool al = (uintptr_t)A0 % 16 == 0 && (uintptr_t)A1 % 16 == 0 && d0 % 4 == 0 && d1 % 4 == 0;
  if (al && T0 >= 16 && T1 >= 16) return 4;
  return T0 >= 4 && T1 >= 4 ? 1 : 0;
}

static bool dma_fits(int d0, int d1, int k, int nb, int vec) {
  if (nb != 2 || vec == 0) return false;
  if (k > 16) return false;   // two k-tiles would not fit the registers
  const int TT = (d0 + 15) / 16 + (d1 + 15) / 16;
  if (TT > kDmaMaxTiles) return false;
  return dma_lds_bytes(d0, d1) <= (size_t)kPassLds + 8 * 1024;
}

// cols: columns of a staged row (16 a tile).
template <class CT> static size_t pass_lds_bytes(int cols, int NT) {
  return ((size_t)16 * pass_pitch(cols) + (size_t)kPassWaves * NT * 256 + (size_t)NT * 272) * sizeof(CT);
}

// Counter that the pass reductions of the current gram_pass_run call on
// this host thread bump (null: none).  Set for the length of one call.
static thread_local int* t_pass_ran = nullptr;

// J_b[c][j] = sum over partials, in a fixed order: each of 4 thread groups
// sums a contiguous quarter of the partials, then the quarters are added.
// A pass that ran (no done flag set) also counts itself in *ran when given.
template <class CT>
__global__ void __launch_bounds__(256) k_pass_reduce(const CT* __restrict__ partial, int nparts, int d0, int d1,
                                                     int W_out, double* __restrict__ J0, double* __restrict__ J1,
                                                     const int* __restrict__ done, int* __restrict__ ran) {
  if (done && *done) return;
  if (ran && blockIdx.x == 0 && threadIdx.x == 0) ++*ran;
  __shared__ double q4[4][64];
  const int64_t Dtot = d0 + d1;
  const int64_t count = Dtot * W_out;
  const int grp = threadIdx.x >> 6, lanei = threadIdx.x & 63;
  const int64_t i = blockIdx.x * 64ll + lanei;
  const int per = (nparts + 3) / 4;
  const int z0 = grp * per, z1 = min(nparts, z0 + per);
  double v = 0.0;
  if (i < count) {
    // loads in batches of 16 (all in flight together), added in z order
    int z = z0;
    for (; z + 16 <= z1; z += 16) {
      CT t[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) t[u] = partial[(int64_t)(z + u) * count + i];
#pragma unroll
      for (int u = 0; u < 16; ++u) v += (double)t[u];
    }
    for (; z < z1; ++z) v += (double)partial[(int64_t)z * count + i];
  }
  q4[grp][lanei] = v;
  __syncthreads();
  if (grp == 0 && i < count) {
    const double tot = ((q4[0][lanei] + q4[1][lanei]) + q4[2][lanei]) + q4[3][lanei];
    const int64_t row = i / W_out, col = i % W_out;
    if (row < d0) J0[row * W_out + col] = tot;
    else J1[(row - d0) * W_out + col] = tot;
  }
}

// ------------------------------------------------------------------
// BF16 data with BF16 matrix-core products (FP32 accumulation): the
// low-precision form of the pass, pipelined like k_pass_quad over one loader,
// three producer and eight consumer waves (three waves a SIMD, 168 registers
// each: the consumers hold the 32 x 2048 sums of a CU):
//   * the loader moves rows of R (8, or 16 up to 64 tiles) into a ring of
//     four LDS blocks, 16 bytes a lane, and the last d % 8 columns of a row
//     4 bytes a lane: no column past a view's last is written, so those of
//     its last 32-column tile stay zero (A_1's tiles start on a 32-column
//     boundary);
//   * the producers form P_b = A_b W_b on 16x16x32 products.  32-column tile
//     T belongs to chain T mod 8; a chain's tiles are summed in turn by the
//     matrix cores and the eight chains in order 0 .. 7: chains 0 - 2 by
//     their producer, the others' sums are added by the consumers.  Eight
//     rows fill half the product's rows (the others repeat them);
//   * the consumers round P to BF16 and accumulate J = A^T [P_0 | P_1] for 32
//     columns of A and the 32 of [P_0 | P_1] (16 a view) at a time on
//     32x32x8 products, whose contraction is eight rows of a block; A comes
//     transposed out of LDS (ds_read_b64_tr_b16: a lane's column, four rows).
// Bounds: the row stream (5.3 to 5.7 TB/s) where the loader stays a block
// ahead.  Two views whose widths are both no multiple of 8 have 64 loads a
// block or more with 16 rows, past what bf_wait counts: the loader then waits
// for the block it has just issued, and a step also for a trip to memory
// (52344 x (532 + 348): 3.3 TB/s).
// Measured, us, against eight waves that did both products in turn with A
// read from LDS two bytes a lane: 200000 x (1000 + 1000), k = 10 230 -> 151;
// 100000 x 2000, k = 16 96 -> 71; 52344 x (532 + 348), k = 9 83 -> 28;
// 100000 x (1002 + 998), k = 3 (4-byte loads before) 267 -> 79.
constexpr int kBfProd = 3, kBfCons = 8;
constexpr int kBfThreads = 64 * (kBfProd + kBfCons + 1);
constexpr int kBfChains = 8, kBfParts = 6;   // chain sums a row's element of P is stored as
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct BfGeom {
  int T0, T1, T0p, T1p, TTp;
};
__host__ __device__ inline BfGeom bf_geom(int d0, int d1) {
  BfGeom g;
  g.T0 = (d0 + 15) / 16;
  g.T1 = (d1 + 15) / 16;
  g.T0p = (g.T0 + 1) & ~1;
  g.T1p = (g.T1 + 1) & ~1;
  g.TTp = g.T0p + g.T1p;
  return g;
}

// TPC: 32-column tiles of a chain, and of a consumer.
template <int R_, int TPC_>
struct BfShape {
  static constexpr int R = R_, TPC = TPC_;
  // row pitch in elements, 64 bytes mod 256: rows 0 - 3 of a transposed read
  // and of the producers' 64-byte runs fall on all 64 banks
  static constexpr int PITCH = 32 * kBfChains * TPC + 32;
  static constexpr int BUF = R * PITCH;
  static constexpr int PART = R * 32 * kBfParts;   // floats: [R][32] of four, then [R][32] of two
  static constexpr size_t lds_bytes() { return (size_t)kPipeRing * BUF * 2 + 2 * PART * 4; }
};

// The directions as the producers' operands: lane (l16, g) of 32-column tile T
// takes W[32 T + 8 g + e][l16], e < 8 (zero past d and k; A_1's tiles from
// tiles0 on).
__global__ void k_pack_dir_bf(const double* __restrict__ W0, int d0, const double* __restrict__ W1, int d1, int tiles0,
                              int k, int count, uint16_t* __restrict__ Wp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int e = i & 7, l16 = (i >> 3) & 15, g = (i >> 7) & 3, T = i >> 9;
  const bool b1 = T >= tiles0;
  const int r = 32 * (b1 ? T - tiles0 : T) + 8 * g + e;
  const float v = r < (b1 ? d1 : d0) && l16 < k ? (float)(b1 ? W1 : W0)[(int64_t)r * k + l16] : 0.0f;
  Wp[i] = bf16_rne_bits(v);
}

// The loads of the R rows at a0 (and a1), `left` of them before the end of
// the data (rows past it read zero).  Returns the number in flight.
template <int NB, class S, bool NT>
__device__ __forceinline__ int bf_load(const unsigned short* a0, const unsigned short* a1, int64_t left, int d0, int d1,
                                       int T0p, unsigned short* __restrict__ dst, int lane) {
  int cnt = 0;
#pragma unroll
  for (int v = 0; v < NB; ++v) {
    const int d = v ? d1 : d0, whole = d & ~7, tail = d & 7;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(v ? a1 : a0, left * d * 2);
    unsigned short* dv = dst + (v ? T0p * 16 : 0);
    for (int c0 = 0; c0 < whole; c0 += 512) {
      const int c = c0 + 8 * lane;
      if (c < whole)
#pragma unroll
        for (int r = 0; r < S::R; ++r) dma_row_chunk<4, NT>(rs, (float*)(dv + r * S::PITCH + c0), (r * d + c) * 2);
      cnt += S::R;
    }
    if (tail) {
      if (2 * lane < tail)
#pragma unroll
        for (int r = 0; r < S::R; ++r)
          dma_row_chunk<1>(rs, (float*)(dv + r * S::PITCH + whole), (r * d + whole + 2 * lane) * 2);
      cnt += S::R;
    }
  }
  return cnt;
}

// At most n (a multiple of 8) of this wave's loads outstanding; none past 56.
__device__ __forceinline__ void bf_wait(int n) {
  switch (n) {
#define SRP_VM(N) case N: __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8)); break;
    SRP_VM(8) SRP_VM(16) SRP_VM(24) SRP_VM(32) SRP_VM(40) SRP_VM(48) SRP_VM(56)
#undef SRP_VM
    default: __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));
  }
}

// A producer's chains (NCH from c0 on) of P for the block in xs.
template <class S, int NB, int NCH>
__device__ __forceinline__ void bf_produce(const unsigned short* __restrict__ xs, float* __restrict__ part, int lane,
                                           int c0, int tiles0, const bf16x8_t (&wreg)[NCH][S::TPC]) {
  constexpr int R = S::R, TPC = S::TPC;
  const int g = lane >> 4, l16 = lane & 15;
  const unsigned short* xp = xs + (l16 & (R - 1)) * S::PITCH + 8 * g;
  f32x4 sum[NB];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    f32x4 pacc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) pacc[b] = f32x4{0, 0, 0, 0};
    // four operands read ahead of their products; past the last tile zeros
    // meet zeros
    constexpr int B = TPC < 4 ? TPC : 4;
#pragma unroll
    for (int i0 = 0; i0 < TPC; i0 += B) {
      bf16x8_t a[B];
#pragma unroll
      for (int u = 0; u < B; ++u) a[u] = *reinterpret_cast<const bf16x8_t*>(xp + 32 * (c0 + c + kBfChains * (i0 + u)));
#pragma unroll
      for (int u = 0; u < B; ++u) {
        if (NB == 2 && c0 + c + kBfChains * (i0 + u) >= tiles0)
          pacc[NB - 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], wreg[c][i0 + u], pacc[NB - 1], 0, 0, 0);
        else pacc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], wreg[c][i0 + u], pacc[0], 0, 0, 0);
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (c0 == 0 && c > 0) sum[b] += pacc[b];   // chains 0 - 2: one partial
      else sum[b] = pacc[b];
      // partial 0 is chains 0 - 2, partial m > 0 chain m + 2
      const int m = c0 == 0 ? (c == 2 ? 0 : -1) : c0 + c - 2;
      if (m >= 0 && 4 * g < R) {
        float* pw = part + (m < 4 ? m : R * 32 * 4 + m - 4);
        const int st = m < 4 ? 4 : 2;
#pragma unroll
        for (int r = 0; r < 4; ++r) pw[((4 * g + r) * 32 + 16 * b + l16) * st] = sum[b][r];
      }
    }
  }
}

// A consumer's step: J += A^T [P_0 | P_1] over tiles wj, wj + 8, ...
template <class S, int NB>
__device__ __forceinline__ void bf_consume(const unsigned short* __restrict__ xs, const float* __restrict__ part,
                                           int wj, int lane, f32x16 (&acc)[S::TPC]) {
  const int n = lane & 31, h = lane >> 5;
  // lane's piece of a transposed read: row 4 h + (lane % 16) / 4 of eight,
  // four columns
  const unsigned short* xr = xs + (4 * h + ((lane & 15) >> 2)) * S::PITCH + 16 * ((lane >> 4) & 1) + 4 * (lane & 3) +
                             32 * wj;
#pragma unroll
  for (int q = 0; q < S::R / 8; ++q) {   // eight rows at a time
    s16x4_t a[S::TPC], pb;
#pragma unroll
    for (int i = 0; i < S::TPC; ++i)
      a[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4_t*)(xr + 8 * q * S::PITCH + 32 * kBfCons * i));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int el = (8 * q + 4 * h + e) * 32 + n;
      const float4 u = *reinterpret_cast<const float4*>(part + el * 4);
      const float2 v = *reinterpret_cast<const float2*>(part + S::R * 32 * 4 + el * 2);
      const float x = ((((u.x + u.y) + u.z) + u.w) + v.x) + v.y;
      pb[e] = NB == 2 || n < 16 ? __builtin_bit_cast(short, (__bf16)x) : (short)0;
    }
#pragma unroll
    for (int i = 0; i < S::TPC; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[i], pb, acc[i], 0, 0, 0);
  }
}

template <int NB, int R_, int TPC_>
__global__ void __launch_bounds__(kBfThreads) k_pass_bf(const unsigned short* __restrict__ A0,
                                                        const unsigned short* __restrict__ A1, int64_t n, int d0,
                                                        int d1, int k, const bf16x8_t* __restrict__ Wp, int nrb,
                                                        float* __restrict__ partial, const int* __restrict__ done) {
  if (done && *done) return;
  using S = BfShape<R_, TPC_>;
  constexpr int R = S::R, TPC = S::TPC;
  extern __shared__ unsigned short bsm[];
  float* parts = reinterpret_cast<float*>(bsm + kPipeRing * S::BUF);
  const BfGeom G = bf_geom(d0, NB == 2 ? d1 : 0);
  const int tiles = G.TTp / 2, tiles0 = G.T0p / 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // columns no load writes stay zero
  for (int e = tid; e < kPipeRing * S::BUF / 2; e += kBfThreads) reinterpret_cast<uint32_t*>(bsm)[e] = 0;
  __syncthreads();
  // this workgroup's blocks: pairs of neighbours, as in k_pass_quad
  const int pairs = (nrb + 1) / 2, mine = (pairs - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  const int nst = 2 * mine - ((nrb & 1) && (pairs - 1) % (int)gridDim.x == (int)blockIdx.x ? 1 : 0);
  if (w == kBfProd + kBfCons) {
    auto stream = [&](auto nt_) __attribute__((always_inline)) {
      int64_t row = (int64_t)blockIdx.x * 2 * R;
      auto load = [&](int i) __attribute__((always_inline)) {   // block i, at `row`
        const int cnt = bf_load<NB, S, decltype(nt_)::value>(A0 + row * d0, NB == 2 ? A1 + row * d1 : nullptr, n - row,
                                                             d0, NB == 2 ? d1 : 0, G.T0p, bsm + (i & 3) * S::BUF, lane);
        row += (i & 1) ? (2ll * gridDim.x - 1) * R : R;
        return cnt;
      };
      load(0);
      bf_wait(nst > 1 ? load(1) : 0);   // block 0 has landed
      lds_only_barrier();
      for (int i = 0; i <= nst; ++i) {
        bf_wait(i + 2 < nst ? load(i + 2) : 0);   // block i + 1 has landed; block i + 2 stays in flight
        lds_only_barrier();
      }
    };
    // non-temporal past the memory-side cache, as in k_pass_quad
    if (n * (d0 + (NB == 2 ? d1 : 0)) * 2 > (256ll << 20)) stream(std::integral_constant<bool, true>{});
    else stream(std::integral_constant<bool, false>{});
  } else if (w < kBfProd) {
    auto produce = [&](auto c0_, auto nch_) __attribute__((always_inline)) {
      constexpr int C0 = decltype(c0_)::value, NCH = decltype(nch_)::value;
      bf16x8_t wreg[NCH][TPC];
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int i = 0; i < TPC; ++i) {
          const int T = C0 + c + kBfChains * i;
          wreg[c][i] = bf16x8_t{};
          if (T < tiles) wreg[c][i] = Wp[T * 64 + lane];
        }
      lds_only_barrier();
      for (int i = 0; i <= nst; ++i) {
        if (i < nst)
          bf_produce<S, NB, NCH>(bsm + (i & 3) * S::BUF, parts + (i & 1) * S::PART, lane, C0, tiles0, wreg);
        lds_only_barrier();
      }
    };
    if (w == 0) produce(std::integral_constant<int, 0>{}, std::integral_constant<int, 3>{});
    else if (w == 1) produce(std::integral_constant<int, 3>{}, std::integral_constant<int, 3>{});
    else produce(std::integral_constant<int, 6>{}, std::integral_constant<int, 2>{});
  } else {
    const int wj = w - kBfProd;
    f32x16 acc[TPC];
#pragma unroll
    for (int i = 0; i < TPC; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    lds_only_barrier();
    lds_only_barrier();   // the producers' step 0
    for (int i = 0; i < nst; ++i) {
      bf_consume<S, NB>(bsm + (i & 3) * S::BUF, parts + (i & 1) * S::PART, wj, lane, acc);
      lds_only_barrier();
    }
    // this workgroup's partial (rows = concatenated columns of A, columns =
    // [P_0 | P_1]); lane: column lane % 32 of the products, rows 8 (r / 4) +
    // 4 (lane / 32) + r % 4
    const int W_out = NB * k, v = (lane & 31) >> 4, col = lane & 15;
    float* out = partial + (int64_t)blockIdx.x * (d0 + (NB == 2 ? d1 : 0)) * W_out + v * k + col;
    if (v < NB && col < k)
#pragma unroll
      for (int i = 0; i < TPC; ++i) {
        const int T = wj + kBfCons * i;
        const bool b1 = NB == 2 && T >= tiles0;
        const int row0 = 32 * (b1 ? T - tiles0 : T) + 4 * (lane >> 5), d = b1 ? d1 : d0;
        if (T < tiles)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r / 4) + r % 4;
            if (row < d) out[(int64_t)((b1 ? d0 : 0) + row) * W_out] = acc[i][r];
          }
      }
  }
}

// The BF16 pass takes rows of whole dwords on 4-byte boundaries, views of at
// least 113 columns (narrower ones keep the FP32 arithmetic of k_pass) and
// at most 128 tiles of 16 columns, each view's count rounded up to even.
static bool bf_widths_ok(int d0, int d1, int nb) {
  auto ok = [](int d) { return d % 2 == 0 && (d + 15) / 16 >= 8; };
  return ok(d0) && (nb == 1 || ok(d1));
}
static bool bf_aligned(const void* A0, const void* A1) { return (uintptr_t)A0 % 4 == 0 && (uintptr_t)A1 % 4 == 0; }

static bool bf_fits(int d0, int d1, int k, int nb) {
  return k <= 16 && bf_geom(d0, nb == 2 ? d1 : 0).TTp <= kDmaMaxTiles;
}

template <int NB, int R, int TPC>
static int pass_launch_bf(const unsigned short* A0, const unsigned short* A1, int64_t n, int d0, int d1, int k,
                          const double* W0, const double* W1, double* J0, double* J1, const int* done, Arena& ws,
                          hipStream_t st, hipEvent_t before_pass, hipEvent_t after_pass) {
  using S = BfShape<R, TPC>;
  static_assert(S::lds_bytes() <= 160 * 1024, "the ring and the partials fit a CU's LDS");
  const int nrb = (int)((n + R - 1) / R);
  // at least 4 blocks per workgroup (fewer partials to add for short data)
  const int grid = std::max(1, std::min(num_cus(), (nrb + 3) / 4));
  const int Dtot = d0 + (NB == 2 ? d1 : 0);
  const BfGeom G = bf_geom(d0, NB == 2 ? d1 : 0);
  const int WN = G.TTp / 2 * 512;
  uint16_t* Wp = ws.take<uint16_t>(WN);
  float* part = ws.take<float>((size_t)grid * Dtot * NB * k);
  if (!Wp || !part) { set_error("gram_pass: workspace too small"); return SRP_ENOMEM; }
  hipLaunchKernelGGL(k_pack_dir_bf, dim3(WN / 256), dim3(256), 0, st, W0, d0, W1, NB == 2 ? d1 : 0, G.T0p / 2, k, WN,
                     Wp);
  SRP_LAUNCH_CHECK();
  SRP_TRY(allow_dynamic_lds((const void*)k_pass_bf<NB, R, TPC>, S::lds_bytes()));
  if (before_pass) SRP_HIP(hipEventRecord(before_pass, st));
  hipLaunchKernelGGL((k_pass_bf<NB, R, TPC>), dim3(grid), dim3(kBfThreads), S::lds_bytes(), st, A0, A1, n, d0,
                     NB == 2 ? d1 : 0, k, reinterpret_cast<const bf16x8_t*>(Wp), nrb, part, done);
  SRP_LAUNCH_CHECK();
  if (after_pass) SRP_HIP(hipEventRecord(after_pass, st));
  const int64_t count = (int64_t)Dtot * NB * k;
  hipLaunchKernelGGL((k_pass_reduce<float>), dim3((unsigned)((count + 63) / 64)), dim3(256), 0, st, part, grid, d0,
                     NB == 2 ? d1 : 0, NB * k, J0, J1, done, t_pass_ran);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

static int pass_dispatch_bf(const unsigned short* A0, const unsigned short* A1, int64_t n, int d0, int d1, int k,
                            const double* W0, const double* W1, double* J0, double* J1, const int* done, Arena& ws,
                            hipStream_t st, hipEvent_t ev0, hipEvent_t ev) {
  const int TTp = bf_geom(d0, A1 ? d1 : 0).TTp;
#define SRP_BF_CASE(NB_, TT_, R_, TPC_)                                                                         \
  if (TTp <= TT_) return pass_launch_bf<NB_, R_, TPC_>(A0, A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, ev0, ev);
  if (A1) {
    SRP_BF_CASE(2, 32, 16, 2) SRP_BF_CASE(2, 64, 16, 4) SRP_BF_CASE(2, 128, 8, 8)
  } else {
    SRP_BF_CASE(1, 32, 16, 2) SRP_BF_CASE(1, 64, 16, 4) SRP_BF_CASE(1, 128, 8, 8)
  }
#undef SRP_BF_CASE
  set_error("gram_pass: no BF16 pass instance for %d tiles", TTp);
  return SRP_EINVAL;
}

int pass_limits_ok(int dtype, int compute, int d0, int d1, int k, int nblocks) {
  if (compute == SRP_BF16) {
    if (dtype != SRP_BF16 || k > 16) return 0;
    if (bf_fits(d0, d1, k, nblocks)) return 1;
    return pass_limits_ok(SRP_BF16, SRP_F32, d0, d1, k, nblocks);   // the FP32-arithmetic pass takes it
  }
  const int D = d0 + (nblocks == 2 ? d1 : 0);
  const bool f64 = (compute == SRP_F64);
  if (dtype == SRP_F64 && !f64) return 0;
  if (nblocks == 2 && k > 16) return 0;
  if (nblocks == 1 && k > 32) return 0;
  const int NT = nblocks * ((k + 15) / 16);
  if (f64) {
    if (D > PassCfg<double>::dmax || pass_lds_bytes<double>(D, NT) > (size_t)kPassLds) return 0;
  } else {
    if (D > PassCfg<float>::dmax || pass_lds_bytes<float>(D, NT) > (size_t)kPassLds) return 0;
  }
  return 1;
}

// Number of row groups (each served by kPassSplit workgroups); a multiple
// of the XCD count so that the pair of a group shares an XCD.
static int pass_groups(int64_t n) {
  const int64_t nrb = (n + 15) / 16;
  int64_t g = num_cus() / kPassSplit;
  if (g > nrb) g = nrb;
  g = ((g + kXcds - 1) / kXcds) * kXcds;
  if (g < kXcds) g = kXcds;
  return (int)g;
}

size_t pass_ws_bytes(int64_t n, int d0, int d1, int k, int compute) {
  const size_t cs = compute == SRP_F64 ? 8 : 4;
  const int KT = (k + 15) / 16;
  const int nb = d1 > 0 ? 2 : 1;
  const size_t D = (size_t)d0 + (nb == 2 ? d1 : 0);
  const size_t wp = (((size_t)(d0 + 15) / 16 * 16) + ((size_t)(d1 + 15) / 16 * 16)) * KT * 16 * cs;
  const size_t slots = std::max<size_t>((size_t)pass_groups(n) * kPassSplit, (size_t)num_cus());
  return ((wp + 1023) & ~size_t(255)) + ((slots * D * nb * k * cs + 255) & ~size_t(255));
}

template <class DT, class CT, int NB, int KT>
static int pass_launch(const DT* A0, const DT* A1, int64_t n, int d0, int d1, int k, const double* W0,
                       const double* W1, double* J0, double* J1, const int* done, Arena& ws, hipStream_t st,
                       hipEvent_t before_pass, hipEvent_t after_pass) {
  const int dp0 = (d0 + 15) / 16 * 16, dp1 = NB == 2 ? (d1 + 15) / 16 * 16 : 0;
  const int KP = KT * 16;
  CT* Wp0 = ws.take<CT>((size_t)dp0 * KP);
  CT* Wp1 = NB == 2 ? ws.take<CT>((size_t)dp1 * KP) : nullptr;
  const int groups = pass_groups(n);
  const int grid = groups * kPassSplit;
  const int Dtot = d0 + (NB == 2 ? d1 : 0);
  CT* part = ws.take<CT>((size_t)groups * Dtot * NB * k);
  if (!Wp0 || !part || (NB == 2 && !Wp1)) { set_error("gram_pass: workspace too small"); return SRP_ENOMEM; }
  SRP_TRY(pack_dirs<CT>(W0, d0, dp0, Wp0, W1, d1, dp1, Wp1, k, KP, st));
  const int nrb = (int)((n + 15) / 16);
  const size_t lds = pass_lds_bytes<CT>(dp0 + dp1, NB * KT);
  constexpr int TM = PassCfg<CT>::dmax / 16;
  auto launch = [&](auto tmax) -> int {
    constexpr int T = decltype(tmax)::value;
    SRP_TRY(allow_dynamic_lds((const void*)k_pass<DT, CT, NB, KT, T>, kLdsBytes));
    if (before_pass) SRP_HIP(hipEventRecord(before_pass, st));
    hipLaunchKernelGGL((k_pass<DT, CT, NB, KT, T>), dim3(grid), dim3(kPassThreads), lds, st, A0, A1, n, d0,
                       NB == 2 ? d1 : 0, k, Wp0, Wp1, nrb, part, done);
    SRP_LAUNCH_CHECK();
    return SRP_OK;
  };
  if (NB == 2 && (dp0 + dp1) / 16 > TM) SRP_TRY(launch(std::integral_constant<int, TM + (NB == 2 ? 1 : 0)>{}));
  else SRP_TRY(launch(std::integral_constant<int, TM>{}));
  if (after_pass) SRP_HIP(hipEventRecord(after_pass, st));
  const int64_t count = (int64_t)Dtot * NB * k;
  hipLaunchKernelGGL((k_pass_reduce<CT>), dim3((unsigned)((count + 63) / 64)), dim3(256), 0, st, part, groups, d0,
                     NB == 2 ? d1 : 0, NB * k, J0, J1, done, t_pass_ran);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

template <int TPB, int VEC>
static int pass_launch_dma(const float* A0, const float* A1, int64_t n, int d0, int d1, int k, const double* W0,
                           const double* W1, double* J0, double* J1, const int* done, Arena& ws, hipStream_t st,
                           hipEvent_t before_pass, hipEvent_t after_pass) {
  const int dp0 = (d0 + 15) / 16 * 16, dp1 = (d1 + 15) / 16 * 16;
  const int KP = 16;
  float* Wp0 = ws.take<float>((size_t)dp0 * KP);
  float* Wp1 = ws.take<float>((size_t)dp1 * KP);
  const int nrb = (int)((n + kDmaRows - 1) / kDmaRows);
  // at least 4 blocks per workgroup (fewer partials to add for short data)
  const int grid = std::max(1, std::min(num_cus(), (nrb + 3) / 4));
  const int Dtot = d0 + d1;
  float* part = ws.take<float>((size_t)grid * Dtot * 2 * k);
  if (!Wp0 || !Wp1 || !part) { set_error("gram_pass: workspace too small"); return SRP_ENOMEM; }
  SRP_TRY(pack_dirs<float>(W0, d0, dp0, Wp0, W1, d1, dp1, Wp1, k, KP, st));
  const size_t lds = dma_lds_bytes(d0, d1);
  SRP_TRY(allow_dynamic_lds((const void*)k_pass_dma<TPB, VEC>, kPassLds + 8 * 1024));
  if (before_pass) SRP_HIP(hipEventRecord(before_pass, st));
  hipLaunchKernelGGL((k_pass_dma<TPB, VEC>), dim3(grid), dim3(kF32Threads), lds, st, A0, A1, n, d0,
                     d1, k, Wp0, Wp1, nrb, part, done);
  SRP_LAUNCH_CHECK();
  if (after_pass) SRP_HIP(hipEventRecord(after_pass, st));
  const int64_t count = (int64_t)Dtot * 2 * k;
  hipLaunchKernelGGL((k_pass_reduce<float>), dim3((unsigned)((count + 63) / 64)), dim3(256), 0, st, part, grid, d0,
                     d1, 2 * k, J0, J1, done, t_pass_ran);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

static int pass_dispatch_dma(const float* A0, const float* A1, int64_t n, int d0, int d1, int k, const double* W0,
                             const double* W1, double* J0, double* J1, const int* done, Arena& ws, hipStream_t st,
                             hipEvent_t ev0, hipEvent_t ev) {
  const int vec = dma_vec(A0, A1, d0, d1);
  const int slots = dma_slots(d0, d1);
#define SRP_DMA_CASE(TPB_)                                                                             \
  if (slots == TPB_)                                                                                   \
    return vec == 4 ? pass_launch_dma<TPB_, 4>(A0, A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, ev0, ev) \
                    : pass_launch_dma<TPB_, 1>(A0, A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, ev0, ev);
  SRP_DMA_CASE(6) SRP_DMA_CASE(8)
#undef SRP_DMA_CASE
  set_error("gram_pass: no DMA pass instance for %d tile slots", slots);
  return SRP_EINVAL;
}

// The pipelined pass (k_pass_quad): rows of a block for the tiles of
// [A_0 | A_1], 0 where it has no instance.  Up to 64 tiles two views take
// k <= 16; beyond, the consumers' registers hold at most five 4-column
// groups of sums (two views: k <= 10, one: k <= 20), and with a view past 64
// tiles the producers' hold four (k <= 8; with five they spill: 100000 x
// (1500 + 300), k = 10 took 314 us, k_pass_dma 262).
static int pipe_rows(int d0, int d1, int k, int nb) {
  const int T0 = (d0 + 15) / 16, T1 = nb == 2 ? (d1 + 15) / 16 : 0, TT = T0 + T1;
  const int c4 = (nb * k + 3) / 4;
  // views under four tiles leave most of a producer's groups empty
  if (k < 1 || TT > 128 || T0 < 4 || (nb == 2 && T1 < 4)) return 0;
  const int rows = TT <= 32 ? 16 : TT <= 64 ? 8 : 4;
  const int most = nb == 1 ? 5 : rows > 4 ? 8 : std::max(T0, T1) <= 64 ? 5 : 4;
  return c4 <= most ? rows : 0;
}

template <int NV, int R, int C4, int PG>
static int pass_launch_pipe(const float* A0, const float* A1, int64_t n, int d0, int d1, int k, const double* W0,
                            const double* W1, double* J0, double* J1, const int* done, Arena& ws, hipStream_t st,
                            hipEvent_t before_pass, hipEvent_t after_pass) {
  using S = PipeShape<NV, R, C4, PG>;
  static_assert(S::lds_bytes() <= 160 * 1024, "the ring and the partials fit a CU's LDS");
  const int nrb = (int)((n + S::R - 1) / S::R);
  // at least 4 blocks per workgroup (fewer partials to add for short data)
  const int grid = std::max(1, std::min(num_cus(), (nrb + 3) / 4));   // at most one per pair of blocks
  const int Dtot = d0 + (NV == 2 ? d1 : 0);
  float* part = ws.take<float>((size_t)grid * Dtot * NV * k);
  if (!part) { set_error("gram_pass: workspace too small"); return SRP_ENOMEM; }
  SRP_TRY(allow_dynamic_lds((const void*)k_pass_quad<NV, R, C4, PG>, S::lds_bytes()));
  if (before_pass) SRP_HIP(hipEventRecord(before_pass, st));
  hipLaunchKernelGGL((k_pass_quad<NV, R, C4, PG>), dim3(grid), dim3(kF32Threads), S::lds_bytes(), st, A0, A1, n,
                     d0, d1, k, W0, W1, nrb, part, done);
  SRP_LAUNCH_CHECK();
  if (after_pass) SRP_HIP(hipEventRecord(after_pass, st));
  const int64_t count = (int64_t)Dtot * NV * k;
  hipLaunchKernelGGL((k_pass_reduce<float>), dim3((unsigned)((count + 63) / 64)), dim3(256), 0, st, part, grid, d0,
                     NV == 2 ? d1 : 0, NV * k, J0, J1, done, t_pass_ran);
  SRP_LAUNCH_CHECK();
  return SRP_OK;
}

static int pass_dispatch_pipe(const float* A0, const float* A1, int64_t n, int d0, int d1, int k, const double* W0,
                              const double* W1, double* J0, double* J1, const int* done, Arena& ws, hipStream_t st,
                              hipEvent_t ev0, hipEvent_t ev) {
  const int nb = A1 ? 2 : 1, c4 = (nb * k + 3) / 4;
  int rows = pipe_rows(d0, d1, k, nb);
  // short data: smaller blocks for more workgroups (a workgroup takes at
  // least four blocks: 1500 x (301 + 203), k = 8 takes 15.3 us with 4 rows a
  // block, 18.4 with 16; 3000 x (400 + 300), k = 4 16.8 with 4, 15.7 with 8)
  while (c4 <= 5 && rows > 4 && n < (int64_t)rows * num_cus()) rows /= 2;
  // groups of the busiest producer: a quarter of the wider view's 4-tile
  // groups with two views, an eighth with one
  const int tmax = (std::max(d0, nb == 2 ? d1 : 0) + 15) / 16;
  const int pg = ((tmax + 3) / 4 + 8 / nb - 1) / (8 / nb);
#define SRP_PIPE_CASE(NV_, R_, C4_, PG_)                                                                         \
  if (nb == NV_ && rows == R_ && c4 == C4_ && pg <= PG_)                                                         \
    return pass_launch_pipe<NV_, R_, C4_, PG_>(A0, A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, ev0, ev);
#define SRP_PIPE_FIVE(NV_, R_, PG_)                                                                              \
  SRP_PIPE_CASE(NV_, R_, 1, PG_) SRP_PIPE_CASE(NV_, R_, 2, PG_) SRP_PIPE_CASE(NV_, R_, 3, PG_)                   \
  SRP_PIPE_CASE(NV_, R_, 4, PG_) SRP_PIPE_CASE(NV_, R_, 5, PG_)
  SRP_PIPE_FIVE(1, 16, 1)
  SRP_PIPE_FIVE(1, 8, 1) SRP_PIPE_FIVE(1, 8, 2)
  SRP_PIPE_FIVE(1, 4, 1) SRP_PIPE_FIVE(1, 4, 2) SRP_PIPE_FIVE(1, 4, 4)
  SRP_PIPE_FIVE(2, 16, 1) SRP_PIPE_FIVE(2, 16, 2)
  SRP_PIPE_FIVE(2, 8, 1) SRP_PIPE_FIVE(2, 8, 2) SRP_PIPE_FIVE(2, 8, 4)
  SRP_PIPE_FIVE(2, 4, 1) SRP_PIPE_FIVE(2, 4, 2) SRP_PIPE_FIVE(2, 4, 4)
  SRP_PIPE_CASE(2, 4, 1, 8) SRP_PIPE_CASE(2, 4, 2, 8) SRP_PIPE_CASE(2, 4, 3, 8) SRP_PIPE_CASE(2, 4, 4, 8)
  SRP_PIPE_CASE(2, 16, 6, 2) SRP_PIPE_CASE(2, 16, 7, 2) SRP_PIPE_CASE(2, 16, 8, 2)
  SRP_PIPE_CASE(2, 8, 6, 2) SRP_PIPE_CASE(2, 8, 7, 2) SRP_PIPE_CASE(2, 8, 8, 2)
  SRP_PIPE_CASE(2, 8, 6, 4) SRP_PIPE_CASE(2, 8, 7, 4) SRP_PIPE_CASE(2, 8, 8, 4)
#undef SRP_PIPE_FIVE
#undef SRP_PIPE_CASE
  set_error("gram_pass: no pipelined pass instance for %d rows, k = %d", rows, k);
  return SRP_EINVAL;
}

template <class DT, class CT>
static int pass_dispatch_k(const DT* A0, const DT* A1, int64_t n, int d0, int d1, int k, const double* W0,
                           const double* W1, double* J0, double* J1, const int* done, Arena& ws, hipStream_t st,
                           hipEvent_t ev0, hipEvent_t ev) {
  if (A1) return pass_launch<DT, CT, 2, 1>(A0, A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, ev0, ev);
  if (k <= 16) return pass_launch<DT, CT, 1, 1>(A0, A1, n, d0, 0, k, W0, W1, J0, J1, done, ws, st, ev0, ev);
  return pass_launch<DT, CT, 1, 2>(A0, A1, n, d0, 0, k, W0, W1, J0, J1, done, ws, st, ev0, ev);
}

// Name of the pass kernel gram_pass_run launches for a shape, for rows
// that start on 16-byte boundaries (the row alignment only changes the
// load width), or nullptr outside the limits.
const char* gram_pass_kernel_name(int dtype, int compute, int d0, int d1, int k) {
  const int nb = d1 > 0 ? 2 : 1;
  if (nb == 1) d1 = 0;
  if (!pass_limits_ok(dtype, compute, d0, d1, k, nb)) return nullptr;
  const int T0 = (d0 + 15) / 16, T1 = nb == 2 ? (d1 + 15) / 16 : 0;
  const bool al = d0 % 4 == 0 && (nb == 1 || d1 % 4 == 0);
  if (compute == SRP_BF16) {
    if (dtype != SRP_BF16) return nullptr;
    return bf_widths_ok(d0, d1, nb) && bf_fits(d0, d1, k, nb) ? "k_pass_bf" : "k_pass";
  }
  if (compute == SRP_F32 && dtype == SRP_F32) {
    const int vec = (al && T0 >= 16 && (nb == 1 || T1 >= 16)) ? 4 : (T0 >= 4 && (nb == 1 || T1 >= 4)) ? 1 : 0;
    if (pipe_rows(d0, d1, k, nb)) return nb == 1 ? "k_pass_quad1" : "k_pass_quad";
    if (dma_fits(d0, d1, k, nb, vec)) return "k_pass_dma";
  }
  return "k_pass";
}

int gram_pass_run(const void* A0, const void* A1, int dtype, int compute, int64_t n, int d0, int d1, int k,
                  const double* W0, const double* W1, double* J0, double* J1, const int* done, Arena& ws,
                  hipStream_t st, hipEvent_t before_pass, hipEvent_t after_pass, int* ran) {
  struct RanScope {
    explicit RanScope(int* r) { t_pass_ran = r; }
    ~RanScope() { t_pass_ran = nullptr; }
  } ran_scope(ran);
  const int nb = A1 ? 2 : 1;
  if (!pass_limits_ok(dtype, compute, d0, d1, k, nb)) {
    set_error("gram_pass: unsupported shape (d0=%d d1=%d k=%d dtype=%d compute=%d)", d0, d1, k, dtype, compute);
    return SRP_EINVAL;
  }
  if (compute == SRP_BF16) {   // BF16 matrix-core products: BF16 data only
    if (dtype != SRP_BF16) {
      set_error("gram_pass: BF16 products need BF16 data");
      return SRP_EINVAL;
    }
    if (bf_aligned(A0, A1) && bf_widths_ok(d0, d1, nb) && bf_fits(d0, d1, k, nb))
      return pass_dispatch_bf((const unsigned short*)A0, (const unsigned short*)A1, n, d0, d1, k, W0, W1, J0, J1,
                              done, ws, st, before_pass, after_pass);
    // views narrower than one 64-lane row chunk (or rows not 4-byte
    // aligned): the FP32-arithmetic pass reads the same BF16 data
    return pass_dispatch_k<bf16, float>((const bf16*)A0, (const bf16*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st,
                                        before_pass, after_pass);
  }
  if (compute == SRP_F64) {
    switch (dtype) {
      case SRP_F64: return pass_dispatch_k<double, double>((const double*)A0, (const double*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, before_pass, after_pass);
      case SRP_F32: return pass_dispatch_k<float, double>((const float*)A0, (const float*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, before_pass, after_pass);
      case SRP_BF16: return pass_dispatch_k<bf16, double>((const bf16*)A0, (const bf16*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, before_pass, after_pass);
    }
  } else {
    switch (dtype) {
      case SRP_F32:
        if (pipe_rows(d0, d1, k, nb))
          return pass_dispatch_pipe((const float*)A0, (const float*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st,
                                    before_pass, after_pass);
        if (dma_fits(d0, nb == 2 ? d1 : 0, k, nb, dma_vec(A0, A1, d0, d1)))
          return pass_dispatch_dma((const float*)A0, (const float*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st,
                                   before_pass, after_pass);
        return pass_dispatch_k<float, float>((const float*)A0, (const float*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, before_pass, after_pass);
      case SRP_BF16: return pass_dispatch_k<bf16, float>((const bf16*)A0, (const bf16*)A1, n, d0, d1, k, W0, W1, J0, J1, done, ws, st, before_pass, after_pass);
    }
  }
  set_error("gram_pass: bad dtype/compute (%d/%d)", dtype, compute);
  return SRP_EINVAL;
}

}  // namespace srp
