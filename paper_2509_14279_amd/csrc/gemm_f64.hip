// fp32-storage contractions with fp64 arithmetic, any shape and alignment:
//
//     C[i][j] = f( sum_r A(i,r) * B(j,r) + bias[j] )          I x J outputs, reduction length R
//
// the three products of the block and of Linear+ReLU and the feed-forward block's, in every operand orientation.
//
// Bound: the fp64 matrix rate (77 TFLOP/s measured), which v_mfma_f64_16x16x4_f64 shares with the vector ALU: whatever the
// loop does besides MFMAs comes on top.  Hence
//   * an element is widened once, on its way into LDS (which holds doubles), not by each wavefront that reads it;
//   * the loop carries no bounds: rows past the end of an operand are read from its last row (their results are not
//     stored), slices that could reach past a row or the matrix - the last one - are done apart, element by element;
//   * a slice costs a thread two 16-byte loads from pointers that advance by a constant, eight conversions, four LDS
//     writes, and its wavefront 16 MFMAs.
// Workgroup: 256 threads = 4 waves (2 x 2), block tile 64 x 64, wave tile 32 x 32, slices of 16, loads two slices ahead,
// LDS double-buffered with one barrier per slice; four workgroups per compute unit cover each other's latencies.
//
// A compute unit's time is the number of tiles it is dealt.  Whole rounds of 256 tiles are done as they are; the tiles of an
// incomplete last round (or all tiles, where that is estimated to be faster) are split over the reduction in the same launch, leave fp64 sums, and
// a second kernel adds them in order (f64_plan).  Small products are dealt out otherwise (f64_small_unit).
// Measured, us (floor at 77 TFLOP/s): 8192 x 1024 x 1024 251 - 260 (223) for each orientation; 64-wide tiles whose operands
// were widened at every read, with bounds in the loop, took 314 - 325 for 4096 x 1024 x 2048 (now 256 - 281).
#include "common.hip.h"
#include "internal.h"

namespace fdl {
namespace {

enum { F64_STORE = 0, F64_RELU = 1, F64_MASK = 2 };

struct F64Params {
  const float* A; const float* B; float* C;
  const float* bias;       // [J] or null
  const float* aux;        // [I][J] (F64_MASK)
  double* part;            // [split][split tiles][64][64]
  int64_t lda, ldb, I, J, R;
  int64_t rlen;            // reduction length of a part (a multiple of 16)
  int tiles_j;
  int whole;               // tiles done as a whole: the first of them; the others are split
  int parted;              // tiles split
};

typedef __attribute__((ext_vector_type(2))) double f64x2;
typedef float f32x4_e __attribute__((ext_vector_type(4), aligned(4)));

// One operand's 64 x 16 slice.  RC (reduction-contiguous in memory): LDS [64][18] doubles, a thread holds four reduction
// indices of one row; else (row index = reduction index): LDS [16][68] doubles, four consecutive i of one reduction index.
// The pads keep a fragment's 16-byte (8-byte) reads within two lanes per bank.
template <bool RC> struct Side {
  static constexpr int kDoubles = RC ? 64 * 18 : 16 * 68;
  const float* at;         // this thread's chunk of the slice fetched next
  int64_t step;            // elements from slice to slice
  int put;                 // its place in LDS, in doubles
  int get[2];              // the lane's fragments (blocks 0, 1)

  __device__ __forceinline__ void init(const float* base, int64_t ld, int64_t i0, int64_t I, int64_t r0, int tid, int w) {
    const int lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    if (RC) {
      int64_t row = i0 + (tid >> 2);
      row = row < I ? row : I - 1;
      at = base + row * ld + r0 + (tid & 3) * 4;
      step = 16;
      put = (tid >> 2) * 18 + (tid & 3) * 4;
      get[0] = (w * 32 + l16) * 18 + g * 4;
      get[1] = get[0] + 16 * 18;
    } else {
      int64_t col = i0 + (tid & 15) * 4;
      col = col < I ? col : (I - 1) & ~(int64_t)3;
      at = base + (r0 + (tid >> 4)) * ld + col;
      step = 16 * ld;
      put = (tid >> 4) * 68 + (tid & 15) * 4;
      get[0] = g * 4 * 68 + w * 32 + l16;
      get[1] = get[0] + 16;
    }
  }
  __device__ __forceinline__ f32x4_e fetch() const { return *reinterpret_cast<const f32x4_e*>(at); }
  // the chunk of the slice at r0, element by element: zeros past the end of either dimension
  static __device__ __forceinline__ f32x4_e fetch_guarded(const float* base, int64_t ld, int64_t i0, int64_t I, int64_t r0,
                                                          int64_t R, int tid) {
    f32x4_e v;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int64_t i = RC ? i0 + (tid >> 2) : i0 + (tid & 15) * 4 + e;
      const int64_t r = RC ? r0 + (tid & 3) * 4 + e : r0 + (tid >> 4);
      // (unconditional, from the nearest element inside: a load under a condition waits for the one before it)
      const int64_t ic = i < I ? i : I - 1, rc = r < R ? r : R - 1;
      v[e] = base[RC ? ic * ld + rc : rc * ld + ic];
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int64_t i = RC ? i0 + (tid >> 2) : i0 + (tid & 15) * 4 + e;
      const int64_t r = RC ? r0 + (tid & 3) * 4 + e : r0 + (tid >> 4);
      v[e] = i < I && r < R ? v[e] : 0.0f;
    }
    return v;
  }
  __device__ __forceinline__ void stash(double* lds, f32x4_e v) const {
    f64x2 lo, hi;
    lo[0] = (double)v[0]; lo[1] = (double)v[1]; hi[0] = (double)v[2]; hi[1] = (double)v[3];
    *reinterpret_cast<f64x2*>(lds + put) = lo;
    *reinterpret_cast<f64x2*>(lds + put + 2) = hi;
  }
  __device__ __forceinline__ void frag(const double* lds, int a, double (&f)[4]) const {
    if (RC) {
      const f64x2 lo = *reinterpret_cast<const f64x2*>(lds + get[a]), hi = *reinterpret_cast<const f64x2*>(lds + get[a] + 2);
      f[0] = lo[0]; f[1] = lo[1]; f[2] = hi[0]; f[3] = hi[1];
    } else {
#pragma unroll
      for (int s = 0; s < 4; s++) f[s] = lds[get[a] + s * 68];
    }
  }
};

template <int EPI> __device__ __forceinline__ void finish_element(const F64Params& p, int64_t i, int64_t j, double z) {
  if (EPI == F64_MASK) p.C[i * p.J + j] = z > 0.0 ? p.aux[i * p.J + j] : 0.0f;
  else p.C[i * p.J + j] = (float)(EPI == F64_RELU ? (z > 0.0 ? z : 0.0) : z);
}

constexpr int kF64LdsDoubles = 2 * 2 * Side<true>::kDoubles;      // two slices of both operands, the larger layout
inline int f64_units(const F64Params& p, int split) { return (p.whole + 7) / 8 * 8 + p.parted * split; }

// unit `id` of a product (f64_units of them)
template <bool A_RC, bool B_RC, int EPI>
__device__ __forceinline__ void f64_unit(const F64Params& p, const int id, double* smem) {
  typedef Side<A_RC> SA;
  typedef Side<B_RC> SB;
  double* lds[2] = {smem, smem + SA::kDoubles + SB::kDoubles};
  // neighbouring tiles - they share operand panels - on one die (ids are dealt round-robin over 8)
  const int per = (p.whole + 7) / 8;
  const bool parted = id >= per * 8;
  const int unit = id - per * 8;                    // (part, tile) of the split tiles
  const int pt = parted ? unit / p.parted : 0;
  const int tile = parted ? p.whole + unit % p.parted : (id & 7) * per + (id >> 3);
  if (!parted && tile >= p.whole) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wi = wave >> 1, wj = wave & 1;
  const int64_t i0 = (int64_t)(tile / p.tiles_j) * 64, j0 = (int64_t)(tile % p.tiles_j) * 64;
  const int64_t r_begin = parted ? pt * p.rlen : 0;
  const int64_t r_end = parted && r_begin + p.rlen < p.R ? r_begin + p.rlen : p.R;
  // Slices the loop may read with whole vectors: inside the reduction and, where a row is a reduction index and a vector
  // may pass its end into the next row, not with the matrix's last row (a vector passes by at most three elements).
  const bool plain = (A_RC || p.lda >= 4) && (B_RC || p.ldb >= 4);
  const int64_t r_safe = (A_RC && B_RC) || r_end < p.R ? r_end : p.R - 1;
  const int full = plain && r_safe > r_begin ? (int)((r_safe - r_begin) / 16) : 0;

  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 4; r++) acc[a][b][r] = 0.0;
  SA sa; SB sb;
  sa.init(p.A, p.lda, i0, p.I, r_begin, tid, wi);
  sb.init(p.B, p.ldb, j0, p.J, r_begin, tid, wj);
  // the accumulators stay in AGPRs from slice to slice (left to itself the compiler moves all of them to VGPRs and back
  // once per trip through the loop, on the unit that does the products)
  auto pin = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int b = 0; b < 2; b++) asm volatile("" : "+a"(acc[a][b]));
  };
  pin();
  auto multiply = [&](const double* la, const double* lb) __attribute__((always_inline)) {
    double fa[2][4], fb[2][4];
#pragma unroll
    for (int a = 0; a < 2; a++) { sa.frag(la, a, fa[a]); sb.frag(lb, a, fb[a]); }
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a][s], fb[b][s], acc[a][b], 0, 0, 0);
    pin();
  };

  if (full > 0) {
    f32x4_e ra[2], rb[2];
    // (past the last slice the pointers stay: it is fetched again, unused)
    int ahead = 0;
    auto advance = [&]() __attribute__((always_inline)) {
      const bool more = ++ahead < full;
      sa.at += more ? sa.step : 0;
      sb.at += more ? sb.step : 0;
    };
    ra[0] = sa.fetch(); rb[0] = sb.fetch(); advance();
    ra[1] = sa.fetch(); rb[1] = sb.fetch(); advance();
    sa.stash(lds[0], ra[0]); sb.stash(lds[0] + SA::kDoubles, rb[0]);
    __syncthreads();
    auto slice = [&](int k) __attribute__((always_inline)) {      // k: the LDS buffer, a constant once inlined
      ra[k] = sa.fetch(); rb[k] = sb.fetch(); advance();
      multiply(lds[k], lds[k] + SA::kDoubles);
      sa.stash(lds[k ^ 1], ra[k ^ 1]); sb.stash(lds[k ^ 1] + SA::kDoubles, rb[k ^ 1]);
      __syncthreads();
    };
    int s = 0;
    for (; s + 2 <= full; s += 2) { slice(0); slice(1); }
    if (s < full) slice(0);
  }
  for (int64_t r = r_begin + (int64_t)full * 16; r < r_end; r += 16) {
    const f32x4_e va = SA::fetch_guarded(p.A, p.lda, i0, p.I, r, r_end, tid);
    const f32x4_e vb = SB::fetch_guarded(p.B, p.ldb, j0, p.J, r, r_end, tid);
    __syncthreads();
    sa.stash(lds[0], va); sb.stash(lds[0] + SA::kDoubles, vb);
    __syncthreads();
    multiply(lds[0], lds[0] + SA::kDoubles);
  }

  // accumulator register r of lane l: output row 4 r + l / 16, column l % 16
  if (parted) {
    double* out = p.part + ((int64_t)pt * p.parted + (tile - p.whole)) * 4096;
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int b = 0; b < 2; b++)
          out[(wi * 32 + a * 16 + r * 4 + (lane >> 4)) * 64 + wj * 32 + b * 16 + (lane & 15)] = acc[a][b][r];
    return;
  }
#pragma unroll
  for (int b = 0; b < 2; b++) {
    const int64_t j = j0 + wj * 32 + b * 16 + (lane & 15);
    if (j >= p.J) continue;
    const double bias = p.bias != nullptr ? (double)p.bias[j] : 0.0;
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int64_t i = i0 + wi * 32 + a * 16 + r * 4 + (lane >> 4);
        if (i >= p.I) continue;
        finish_element<EPI>(p, i, j, acc[a][b][r] + bias);
      }
  }
}

template <bool A_RC, bool B_RC, int EPI>
__global__ __launch_bounds__(256) void gemm_f64_kernel(F64Params p) {
  __shared__ __attribute__((aligned(16))) double lds[kF64LdsDoubles];
  f64_unit<A_RC, B_RC, EPI>(p, (int)blockIdx.x, lds);
}

// dX = dZ W and dW = dZ^T X side by side in one launch (launch_f64_grads says where).  dW comes
// first (its reduction, over the batch, is usually the longer one).
__global__ __launch_bounds__(256) void gemm_f64_pair_kernel(F64Params dx, F64Params dw, int dw_units) {
  __shared__ __attribute__((aligned(16))) double lds[kF64LdsDoubles];
  const int id = (int)blockIdx.x;
  if (id < dw_units) f64_unit<false, false, F64_STORE>(dw, id, lds);
  else f64_unit<true, false, F64_STORE>(dx, id - dw_units, lds);
}

// ---- small products: 32 x 32 tiles, the reduction dealt over a workgroup's four wavefronts ------------------------------------
// Layers of a few hundred rows and columns have fewer 64 x 64 tiles than compute units, and a split of those leaves sums that another
// launch, of 4 us whatever it does, has to add.  Here a wavefront has the whole tile (2 x 2 blocks) for every fourth step of 16 indices, takes
// its fragments straight from memory, widened in registers, and the four sums meet in LDS, in order: no operand passes through LDS
// and no barrier stands before the end.  Bound: latency - the launch, the first loads, 1024 cycles of MFMA per step.
// 256^3, us, split 64 x 64 tiles / so: step 25.5 / 20.5, Linear+ReLU forward and backward 32.8 / 21.0.
template <bool RC> struct Strip {
  const float* at;         // RC: the lane's row at its first index; else column
  int64_t ld;
  __device__ __forceinline__ void init(const float* base, int64_t ld_, int64_t i, int64_t I, int g) {
    i = i < I ? i : I - 1;                           // (past the end: the last row again, whose results are not stored)
    ld = ld_;
    at = RC ? base + i * ld + g * 4 : base + (int64_t)(g * 4) * ld + i;
  }
  __device__ __forceinline__ f32x4_e fetch(int64_t k) const {
    if (RC) return *reinterpret_cast<const f32x4_e*>(at + k);
    f32x4_e v;
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = at[(k + e) * ld];
    return v;
  }
  // left: indices from the lane's first one to the end
  __device__ __forceinline__ f32x4_e fetch_guarded(int64_t k, int64_t left) const {
    f32x4_e v;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      // (unconditional, from the last index inside)
      const int64_t kk = k + (e < left ? e : left - 1);
      v[e] = at[RC ? kk : kk * ld];
    }
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = e < left ? v[e] : 0.0f;
    return v;
  }
};

constexpr int kSmallTile = 32, kSmallDepth = 4;      // steps a wavefront has in flight
constexpr int kSmallLds = 4 * kSmallTile * (kSmallTile + 1);      // doubles
inline int64_t small_tiles(int64_t I, int64_t J) { return ((I + kSmallTile - 1) / kSmallTile) * ((J + kSmallTile - 1) / kSmallTile); }

template <bool A_RC, bool B_RC, int EPI>
__device__ __forceinline__ void f64_small_unit(const F64Params& p, const int tile, double* smem) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (int64_t)(tile / p.tiles_j) * kSmallTile, j0 = (int64_t)(tile % p.tiles_j) * kSmallTile;
  Strip<A_RC> sa[2]; Strip<B_RC> sb[2];
#pragma unroll
  for (int a = 0; a < 2; a++) {
    sa[a].init(p.A, p.lda, i0 + a * 16 + l16, p.I, g);
    sb[a].init(p.B, p.ldb, j0 + a * 16 + l16, p.J, g);
  }
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 4; r++) acc[a][b][r] = 0.0;
  auto multiply = [&](const f32x4_e (&va)[2], const f32x4_e (&vb)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)va[a][s], (double)vb[b][s], acc[a][b], 0, 0, 0);
  };
  const int64_t full = p.R / 16, rounds = full / (4 * kSmallDepth);
  for (int64_t t = 0; t < rounds; t++) {
    f32x4_e va[kSmallDepth][2], vb[kSmallDepth][2];
#pragma unroll
    for (int u = 0; u < kSmallDepth; u++) {
      const int64_t k = ((t * kSmallDepth + u) * 4 + wave) * 16;
#pragma unroll
      for (int a = 0; a < 2; a++) { va[u][a] = sa[a].fetch(k); vb[u][a] = sb[a].fetch(k); }
    }
    __builtin_amdgcn_sched_barrier(0);               // (all loads first)
#pragma unroll
    for (int u = 0; u < kSmallDepth; u++) multiply(va[u], vb[u]);
  }
  for (int64_t s = rounds * 4 * kSmallDepth + wave; s * 16 < p.R; s += 4) {
    const int64_t k = s * 16, left = p.R - k - g * 4;
    f32x4_e va[2], vb[2];
#pragma unroll
    for (int a = 0; a < 2; a++) {
      if (left >= 4) {
        va[a] = sa[a].fetch(k); vb[a] = sb[a].fetch(k);
      } else {
        va[a] = sa[a].fetch_guarded(k, left); vb[a] = sb[a].fetch_guarded(k, left);
      }
    }
    multiply(va, vb);
  }
  constexpr int kRow = kSmallTile + 1;
  double* mine = smem + wave * kSmallTile * kRow;
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 4; r++) mine[(a * 16 + r * 4 + g) * kRow + b * 16 + l16] = acc[a][b][r];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const int at = e * 256 + (int)threadIdx.x, row = at >> 5, col = at & 31;
    double z = smem[row * kRow + col];
#pragma unroll
    for (int w = 1; w < 4; w++) z += smem[(w * kSmallTile + row) * kRow + col];
    const int64_t i = i0 + row, j = j0 + col;
    if (i < p.I && j < p.J) finish_element<EPI>(p, i, j, z + (p.bias != nullptr ? (double)p.bias[j] : 0.0));
  }
}

template <bool A_RC, bool B_RC, int EPI>
__global__ __launch_bounds__(256) void gemm_f64_small_kernel(F64Params p) {
  __shared__ double smem[kSmallLds];
  f64_small_unit<A_RC, B_RC, EPI>(p, (int)blockIdx.x, smem);
}
// dW, dX and, behind them, the column sums (as f64_finish_kernel's)
__global__ __launch_bounds__(256) void gemm_f64_small_pair_kernel(F64Params dx, F64Params dw, int dw_units, int units, TailSums j) {
  __shared__ double smem[kSmallLds];
  const int id = (int)blockIdx.x;
  if (id >= units) {
    const int cblocks = (int)((j.N + 63) / 64), which = (id - units) / cblocks;
    b2_columns<double, 4>(j.N, j.groups, j.kinds, reinterpret_cast<const double*>(j.colpart), (id - units) % cblocks, which,
                          which == 0 ? j.col_out[0] : (which == 1 ? j.col_out[1] : j.col_out[2]), reinterpret_cast<double (*)[64]>(smem));
  } else if (id < dw_units) {
    f64_small_unit<false, false, F64_STORE>(dw, id, smem);
  } else {
    f64_small_unit<true, false, F64_STORE>(dx, id - dw_units, smem);
  }
}

// the split tiles' outputs: the parts' sums in order, then as above; 1024 elements of a tile from `at`, four per thread
template <int EPI> __device__ __forceinline__ void f64_reduce_tile(const F64Params& p, int split, int t, int at) {
  const int tile = p.whole + t;
  const int64_t i = (int64_t)(tile / p.tiles_j) * 64 + at / 64, j = (int64_t)(tile % p.tiles_j) * 64 + at % 64;
  if (i >= p.I || j >= p.J) return;
  f64x4 z = *reinterpret_cast<const f64x4*>(p.part + (int64_t)t * 4096 + at);
  for (int k = 1; k < split; k++) {
    const f64x4 x = *reinterpret_cast<const f64x4*>(p.part + ((int64_t)k * p.parted + t) * 4096 + at);
#pragma unroll
    for (int e = 0; e < 4; e++) z[e] += x[e];
  }
#pragma unroll
  for (int e = 0; e < 4; e++)
    if (j + e < p.J) finish_element<EPI>(p, i, j + e, z[e] + (p.bias != nullptr ? (double)p.bias[j + e] : 0.0));
}

// four workgroups per tile
template <int EPI>
__global__ __launch_bounds__(256) void f64_reduce_kernel(F64Params p, int split) {
  f64_reduce_tile<EPI>(p, split, (int)blockIdx.x >> 2, ((int)blockIdx.x & 3) * 1024 + (int)threadIdx.x * 4);
}

// The end of a backward pass in one launch: the split tiles of dX and dW, a workgroup per tile, then the column sums
// (j.kinds ceil(N / 64) workgroups, as b2_kernel).
__global__ __launch_bounds__(1024) void f64_finish_kernel(F64Params dx, int split_x, F64Params dw, int split_w, TailSums j) {
  __shared__ double red[16][64];
  int id = (int)blockIdx.x;
  if (id < dw.parted) { f64_reduce_tile<F64_STORE>(dw, split_w, id, (int)threadIdx.x * 4); return; }
  id -= dw.parted;
  if (id < dx.parted) { f64_reduce_tile<F64_STORE>(dx, split_x, id, (int)threadIdx.x * 4); return; }
  id -= dx.parted;
  const int cblocks = (int)((j.N + 63) / 64), which = id / cblocks;
  b2_columns<double>(j.N, j.groups, j.kinds, reinterpret_cast<const double*>(j.colpart), id % cblocks, which,
                     which == 0 ? j.col_out[0] : (which == 1 ? j.col_out[1] : j.col_out[2]), red);
}

// Units that are resident at once (four workgroups on each of 256 compute units): the two gradient products share a launch
// up to here - small layers, which are bound by the launches (256^3: step 45 -> 31 us).  Beyond, each product's own rounds
// are the better schedule (758 x 2048 x 2304: step 398 us with two launches, 427 with one).
constexpr int kF64Resident = 1024;

template <int EPI> void dispatch_f64_main(const GemmDesc& g, const F64Params& p, const F64Split& q, hipStream_t s) {
  if (q.small) {
    auto kern = g.a_rc ? (g.b_rc ? gemm_f64_small_kernel<true, true, EPI> : gemm_f64_small_kernel<true, false, EPI>)
                       : (g.b_rc ? gemm_f64_small_kernel<false, true, EPI> : gemm_f64_small_kernel<false, false, EPI>);
    hipLaunchKernelGGL(kern, dim3((unsigned)small_tiles(p.I, p.J)), dim3(256), 0, s, p);
    return;
  }
  const dim3 grid((unsigned)f64_units(p, q.split));
  auto kern = g.a_rc ? (g.b_rc ? gemm_f64_kernel<true, true, EPI> : gemm_f64_kernel<true, false, EPI>)
                     : (g.b_rc ? gemm_f64_kernel<false, true, EPI> : gemm_f64_kernel<false, false, EPI>);
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, p);
}
template <int EPI> void dispatch_f64(const GemmDesc& g, const F64Params& p, const F64Split& q, hipStream_t s) {
  dispatch_f64_main<EPI>(g, p, q, s);
  if (p.parted > 0) hipLaunchKernelGGL(f64_reduce_kernel<EPI>, dim3((unsigned)p.parted * 4), dim3(256), 0, s, p, q.split);
}

}  // namespace

// Which tiles are split, and into how many parts.  A compute unit works through what it is dealt at about 0.52 us per slice
// of 16, a workgroup alone on it at 0.68, one with little company at 0.58 (0.75 for the stragglers of an incomplete last
// round behind four full ones); the second kernel costs about 4 us, the sums' traffic 6 ns per part of a tile.  Either the tiles of the last round are split,
// or all of them.  Measured, us, without / with the split: 3001 x 771 x 1537 by reduction over 771 (1175 tiles) 143 / 133,
// over 1537 (611) 166 / 140, over 3001 (325, all in 3 parts) 199 / 148; 256^3 (16 tiles, 8 parts) 14.5 / 11; 512^3 24.5 / 16;
// 128 x 4096 x 1024 (32 tiles) 159 / 30.  The plan must not depend on the device: 256 compute units.
constexpr int64_t kF64MaxSmall = 1024;      // 32 x 32 tiles
constexpr int64_t kF64MaxUnits = 2048;      // parts of 32 KB each: at most 64 MB
F64Split f64_plan(int64_t I, int64_t J, int64_t R) {
  const int64_t tiles = ((I + 63) / 64) * ((J + 63) / 64), slices = (R + 15) / 16;
  const int64_t full = tiles / 256, rest = tiles % 256;
  F64Split best = {tiles, 0, 1, 0};
  double best_cost = (double)slices * ((full == 1 && rest == 0 ? 0.68 : full * 0.52) + (rest == 0 ? 0.0 : (full >= 4 ? 0.75 : (full == 0 ? 0.68 : 0.55))));
  for (int split = 2; split <= 16 && split <= slices; split++)
    for (int all = 0; all < 2; all++) {
      const int64_t rounds = all ? 0 : full, parted = tiles - rounds * 256, units = parted * split;
      if (units == 0 || units > kF64MaxUnits || (all && full == 0)) continue;
      const int64_t more = (units + 255) / 256, len = (slices + split - 1) / split;
      double cost = (double)(rounds * slices + more * len) * (rounds + more == 1 ? 0.68 : (rounds == 1 ? 0.58 : 0.52));
      if (rounds > 0 && cost < slices * 0.68) cost = slices * 0.68;
      cost += 4.0 + units * 0.006 + split * 0.15;
      if (cost < (best.split == 1 ? 0.97 : 1.0) * best_cost) { best.whole = rounds * 256; best.parted = parted; best.split = split; best_cost = cost; }
    }
  // 32 x 32 tiles, all of them whole: a step of 64 indices 0.67 us, two tiles on a compute unit twice that.  Inference, us, before / so: 256 x 256
  // x 256 11.2 / 10.7, 512 x 512 x 512 17.3 / 14.6, 500 x 1024 x 512 25.2 / 19.7, 1000 x 200 x 300 18.0 / 14.4; not taken 256 x 1024 x 256 14.1 / 19.2,
  // 1024 x 1024 x 1024 46.2 / 48.8; feed-forward 256 x 512 x 1024 48.4 / 37.2, 100 x 1024 x 2000 63.4 / 52.2.
  const int64_t small = small_tiles(I, J);
  if (small <= kF64MaxSmall && 3.0 + (double)((small + 255) / 256) * (double)((slices + 3) / 4) * 0.67 < 0.92 * best_cost) best.small = 1;
  return best;
}
// Both gradients in 32 x 32 tiles, in one launch with the column sums, which takes the finishing launch away.  Two steps of 16 rows of an
// operand whose rows are reduction indices are 32 loads, so the work of a compute unit (steps of 64) and the longest reduction are
// bounded.  Steps, us, before / so (less what the forward pass gained): 256 x 256 x 256 25.5 / 20.5 (0.6), 300 x 300 x 700 44.3 / 36.6
// (2.7), 1000 x 200 x 300 43.3 / 36.5 (3.6), 256 x 512 x 1024 49.6 / 44.6 (2.3); beyond: 256 x 2048 x 256 41.9 / 44.4 (0), 333 x 777 x 555 53.4 / 52.4 (3.6), 2000 x 128 x 256
// 40.6 / 48.1 (2.3), 1024 x 1024 x 1024 139 / 168.
// Within those bounds a long reduction of few tiles is one wavefront's chain, which a split deals out (Linear+ReLU 24 x 512 x 1024, dX 16 tiles of
// 16 steps: 35.5 split, 42.8 so).  Estimated, us: here 0.5 for each step of the longest unit or 0.74 for each of a compute unit's, 0.24 more
// for these; split 0.7 for each slice of its longest part, 2.7 for 256 parts, 4 for the launch that ends it.  (Fitted to 2727 shapes of 6
// to 16 steps, rms 1.5 us.  On them, whole calls: 0.907 of the split's time on average always so, 0.905 by this rule; 167 and 93 more than 3 % slower
// than split, 1.21 and 1.18 times at most, and by this rule 20 more than 3 % slower than so, 1.10 at most.)
bool f64_small_grads(int64_t M, int64_t K, int64_t N, const F64Split* dx, const F64Split* dw) {
  const int64_t tx = small_tiles(M, K), tw = small_tiles(N, K), sx = (N + 63) / 64, sw = (M + 63) / 64;
  if (!(tx <= kF64MaxSmall && tw <= kF64MaxSmall && sx <= 16 && sw <= 16 && tx + tw <= 768 && tx * sx + tw * sw <= 16 * 256)) return false;
  if (dx == nullptr) return true;
  const F64Split &x = *dx, &w = *dw;
  auto part = [](const F64Split& q, int64_t R) { return (double)((R + 15) / 16) / q.split; };       // slices
  const double longest = (double)(sx > sw ? sx : sw), all = (double)(tx * sx + tw * sw) / 256.0;
  const double px = part(x, N), pw = part(w, M), parts = (x.split > 1 ? (double)x.parted * x.split : 0.0) + (w.split > 1 ? (double)w.parted * w.split : 0.0);
  const double here = (0.5 * longest > 0.74 * all ? 0.5 * longest : 0.74 * all) + 0.24 * all;
  return here < 0.7 * (px > pw ? px : pw) + 2.7 * parts / 256.0 + 4.0;
}
size_t f64_part_bytes(const F64Split& q) { return q.split > 1 ? (size_t)q.parted * q.split * 4096 * 8 : 0; }

// kind 0 plain (bias may be null), 1 max(., 0), 2 aux where the sum is positive else 0; part: f64_part_bytes(q) of scratch,
// q from f64_plan(I, J, R) or {tiles, 0, 1}
static F64Params f64_params(const GemmDesc& g, const F64Split& q, const float* bias, const void* aux, void* C, void* part) {
  F64Params p = {};
  p.A = (const float*)g.A; p.B = (const float*)g.B; p.C = (float*)C; p.bias = bias; p.aux = (const float*)aux;
  p.part = (double*)part;
  p.lda = g.lda; p.ldb = g.ldb; p.I = g.I; p.J = g.J; p.R = g.R;
  p.tiles_j = (int)((g.J + 63) / 64);
  p.whole = (int)q.whole; p.parted = (int)q.parted;
  const int64_t slices = (g.R + 15) / 16;
  if (q.small) { p.whole = p.parted = 0; p.tiles_j = (int)((g.J + kSmallTile - 1) / kSmallTile); return p; }
  p.rlen = (slices + q.split - 1) / q.split * 16;
  return p;
}
void launch_f64(int kind, const GemmDesc& g, const F64Split& q, const float* bias, const void* aux, void* C, void* part,
                hipStream_t s) {
  const F64Params p = f64_params(g, q, bias, aux, C, part);
  if (kind == 1) dispatch_f64<F64_RELU>(g, p, q, s);
  else if (kind == 2) dispatch_f64<F64_MASK>(g, p, q, s);
  else dispatch_f64<F64_STORE>(g, p, q, s);
}

F64Sums launch_f64_parts(const GemmDesc& g, const F64Split& q, const float* bias, void* Z, void* part, hipStream_t s) {
  const F64Params p = f64_params(g, q, bias, nullptr, Z, part);
  dispatch_f64_main<F64_STORE>(g, p, q, s);
  return F64Sums{(const double*)part, bias, (float*)Z, (int64_t)p.parted * 4096, q.split, p.tiles_j};
}

// dX (rows of dZ times W) and dW (columns of dZ times X); launch_f64_grads_finish ends both, and the column sums j, unless both are
// small: then this launch does all
void launch_f64_grads(const F64Grads& a, const TailSums& j, hipStream_t s) {
  const F64Params dx = f64_params(a.dx, a.qx, nullptr, nullptr, a.dX, a.partx), dw = f64_params(a.dw, a.qw, nullptr, nullptr, a.dW, a.partw);
  if (a.qx.small && a.qw.small) {
    const int nw = (int)small_tiles(dw.I, dw.J), nx = (int)small_tiles(dx.I, dx.J);
    const unsigned blocks = (unsigned)(nw + nx) + (unsigned)j.kinds * (unsigned)((j.N + 63) / 64);
    hipLaunchKernelGGL(gemm_f64_small_pair_kernel, dim3(blocks), dim3(256), 0, s, dx, dw, nw, nw + nx, j);
    return;
  }
  const int nw = f64_units(dw, a.qw.split), nx = f64_units(dx, a.qx.split);
  if (nw + nx > kF64Resident) {
    dispatch_f64_main<F64_STORE>(a.dx, dx, a.qx, s);
    dispatch_f64_main<F64_STORE>(a.dw, dw, a.qw, s);
    return;
  }
  hipLaunchKernelGGL(gemm_f64_pair_kernel, dim3((unsigned)(nw + nx)), dim3(256), 0, s, dx, dw, nw);
}
void launch_f64_grads_finish(const F64Grads& a, const TailSums& j, hipStream_t s) {
  if (a.qx.small && a.qw.small) return;
  const F64Params dx = f64_params(a.dx, a.qx, nullptr, nullptr, a.dX, a.partx), dw = f64_params(a.dw, a.qw, nullptr, nullptr, a.dW, a.partw);
  const unsigned blocks = (unsigned)(dx.parted + dw.parted) + (unsigned)j.kinds * (unsigned)((j.N + 63) / 64);
  hipLaunchKernelGGL(f64_finish_kernel, dim3(blocks), dim3(1024), 0, s, dx, a.qx.split, dw, a.qw.split, j);
}

}  // namespace fdl
