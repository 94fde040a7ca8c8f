// bf16 products with few rows: out[m][n] = f(sum_k X[m][k] W[n][k]) for batches below (or not far above) one tile of the
// large contraction kernel - serving a handful of requests, a decoding step of the feed-forward block.
//
// Bound: the weights, which are read once and used for M rows only (2 M flop per byte: at M = 16 a 250th of what would
// keep the matrix pipes busy).  So the kernel is built to keep loads in flight, and nothing else:
//   * a workgroup owns 16 NB output columns and 16 MB rows, and its wavefronts split the reduction among themselves: a
//     4096-wide layer has 256 workgroups of 8 wavefronts, all of them streaming different parts of W;
//   * a lane's MFMA fragment (v_mfma_f32_16x16x32_bf16: row lane % 16, eight reduction indices) is 16 contiguous bytes of
//     a row of X or W, so both operands go straight from global memory into the registers the matrix pipe reads: no LDS
//     tile, no barrier, and U steps of loads in flight per wavefront;
//   * the wavefronts' sums meet in LDS once, at the end, in a fixed order (pairwise), in fp32.
// Measured, M x K x N, us: 16 x 4096 x 4096 11 (3.1 TB/s), 32 rows 15; 16 x 11008 x 4096 23 (3.9 TB/s); gated 16 x 4096 x 11008 37
// (4.9 TB/s; 46 by 64-byte loads).  The 64 x 64 tiles of the generic kernel took 93 us
// for 32 x 4096 x 4096 (64 workgroups, each alone with 256 slices) and 158 for each product of the 16-row block.  Loads of W
// past the caches cost 10 - 20 %; 16 steps in flight gain nothing over 8.
// A compute unit's vector cache has room for 256 lines, which is what limits the loads in flight, X's among them: 1024 lines of either
// matrix take a compute unit 4 us (32 x 4096 x 4096: 7.5 us without the loads of X, 15.2 with).  A fragment's 64-byte pieces of 16 rows
// hold a line for half of its bytes; from kLinesFrom on (which see) a load therefore takes 128 bytes of 8 rows, and lanes exchange what is
// not theirs (as_fragments).
#include "common.hip.h"
#include "internal.h"

#include <type_traits>

namespace fdl {
namespace {

enum { SK_STORE = 0, SK_RELU = 1, SK_MASK = 2, SK_GATE = 3 };

struct SkinnyParams {
  const bf16_t* X; const bf16_t* W; const bf16_t* W2;   // W2: SK_GATE, the up weights
  const float* bias;      // may be null (SK_STORE, SK_RELU, SK_MASK)
  const bf16_t* aux;      // SK_MASK: [M][N]
  bf16_t* out;            // [M][ldo]
  int64_t ldo;
  int64_t K;
  int M, N;
  int mblocks;            // row blocks of 16 MB
};

template <bool AL> __device__ __forceinline__ bf16x8 load8(const bf16_t* p) {
  if constexpr (AL) {
    return *reinterpret_cast<const bf16x8*>(p);
  } else {
    typedef __bf16 bf16x8_u __attribute__((ext_vector_type(8), aligned(2)));
    return *reinterpret_cast<const bf16x8_u*>(p);
  }
}
typedef __attribute__((address_space(1))) const char global_char;
// 16 bytes at a wave-uniform base and a lane's byte offset (one address register)
template <bool AL> __device__ __forceinline__ bf16x8 load8(const bf16_t* base, uint32_t off) {
  asm("" : "+s"(base), "+v"(off));     // (not to be added up ahead of the loop, in twice the registers)
  if constexpr (AL) {
    return *(__attribute__((address_space(1))) const bf16x8*)((global_char*)base + off);
  } else {
    typedef __bf16 bf16x8_u __attribute__((ext_vector_type(8), aligned(2)));
    return *(__attribute__((address_space(1))) const bf16x8_u*)((global_char*)base + off);
  }
}
// v without its first `skip` elements (8 and more: without any), zeros in their place
__device__ __forceinline__ bf16x8 clear_front(bf16x8 v, int skip) {
  if (skip <= 0) return v;
  unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
  x = skip >= 8 ? 0 : x >> (16 * skip) << (16 * skip);
  return __builtin_bit_cast(bf16x8, x);
}

// Two loads of 64 reduction indices of 16 rows: lane l has chunk l / 8 (of 16 bytes) of row l % 8 in lo and of row 8 + l % 8 in hi,
// so that each row's piece is 128 contiguous bytes.  As fragments - lane l: row l % 16, its eight reduction indices the chunk
// 2 (l / 16) in the first, the next one in the second - lanes 8 apart exchange one of their vectors.
__device__ __forceinline__ void as_fragments(bf16x8& lo, bf16x8& hi, bool upper) {
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  i32x4 a = __builtin_bit_cast(i32x4, lo), b = __builtin_bit_cast(i32x4, hi);
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const int give = upper ? a[e] : b[e];
    const int get = __builtin_amdgcn_update_dpp(0, give, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
    if (upper) a[e] = get; else b[e] = get;
  }
  lo = __builtin_bit_cast(bf16x8, a);
  hi = __builtin_bit_cast(bf16x8, b);
}

// AL: K is a multiple of 8 (every row starts on 16 bytes); otherwise the same loads from element-aligned addresses.
// LINES: loads of whole lines, U steps of 64 in flight; otherwise of 64 bytes of 16 rows, U steps of 32.
template <int MB, int NB, int EPI, int WAVES, int U, bool AL, bool LINES>
__global__ __launch_bounds__(64 * WAVES) void gemm_skinny_kernel(SkinnyParams p) {
  constexpr int NMAT = EPI == SK_GATE ? 2 : 1;
  constexpr int NF = NMAT * NB;                      // W fragments per step
  __shared__ f32x4 red[WAVES > 1 ? WAVES / 2 : 1][NF * MB][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  // Row blocks of the same columns are neighbours on one die (workgroup ids are dealt round-robin over 8 dies), so that
  // the weights they share are in its L2 when the second block reads them.
  const int bid = (int)blockIdx.x;
  const int slot = bid >> 3;
  const int strip = (slot / p.mblocks) * 8 + (bid & 7);
  const int n0 = strip * 16 * NB, m0 = (slot % p.mblocks) * 16 * MB;
  if (n0 >= p.N) return;                             // (the grid is rounded up to whole groups of 8)

  // rows past the end of either matrix read the last row; what they contribute is not stored
  f32x4 acc[NF][MB];
#pragma unroll
  for (int f = 0; f < NF; f++)
#pragma unroll
    for (int b = 0; b < MB; b++)
#pragma unroll
      for (int r = 0; r < 4; r++) acc[f][b][r] = 0.0f;

  if constexpr (LINES) {
    const bool upper = (lane & 8) != 0;
    const bf16_t* wb[NF];                            // first row of each block of 16
    const bf16_t* xb[MB];
    uint32_t wo[NF][2], xo[MB][2];                   // the lane's bytes from there (K is at most 2^24)
    auto offset = [&](int h, int last) __attribute__((always_inline)) {
      const int r = h * 8 + (lane & 7);
      return (uint32_t)(r < last ? r : last) * (uint32_t)p.K * 2u + (uint32_t)(lane >> 3) * 16u;
    };
#pragma unroll
    for (int f = 0; f < NF; f++) {
      const int n = n0 + (f % NB) * 16, at = n < p.N ? n : p.N - 1;
      wb[f] = (f < NB ? p.W : p.W2) + (int64_t)at * p.K;
#pragma unroll
      for (int h = 0; h < 2; h++) wo[f][h] = offset(h, p.N - 1 - at);
    }
#pragma unroll
    for (int b = 0; b < MB; b++) {
      const int m = m0 + b * 16, at = m < p.M ? m : p.M - 1;
      xb[b] = p.X + (int64_t)at * p.K;
#pragma unroll
      for (int h = 0; h < 2; h++) xo[b][h] = offset(h, p.M - 1 - at);
    }
    const int full = (int)(p.K >> 6);                  // whole steps of 64
    // C steps from reduction index k0 on; LAST: the first `skip` indices have been counted
    auto steps = [&](auto count, auto last, int64_t k0, int skip) __attribute__((always_inline)) {
      constexpr int C = decltype(count)::value;
      constexpr bool LAST = decltype(last)::value;
      bf16x8 w[C][NF][2], x[C][MB][2];
  #pragma unroll
      for (int u = 0; u < C; u++) {
        const int64_t k = k0 + u * 64;
  #pragma unroll
        for (int h = 0; h < 2; h++) {
  #pragma unroll
          for (int f = 0; f < NF; f++) w[u][f][h] = load8<AL>(wb[f] + k, wo[f][h]);
  #pragma unroll
          for (int b = 0; b < MB; b++) x[u][b][h] = load8<AL>(xb[b] + k, xo[b][h]);
        }
      }
      if (LAST) {
        const int clear = skip - (lane >> 3) * 8;
  #pragma unroll
        for (int h = 0; h < 2; h++) {
  #pragma unroll
          for (int f = 0; f < NF; f++) w[0][f][h] = clear_front(w[0][f][h], clear);
  #pragma unroll
          for (int b = 0; b < MB; b++) x[0][b][h] = clear_front(x[0][b][h], clear);
        }
      }
      __builtin_amdgcn_sched_barrier(0);               // (all loads first: the scheduler would have few in flight to save registers)
  #pragma unroll
      for (int u = 0; u < C; u++) {
  #pragma unroll
        for (int f = 0; f < NF; f++) as_fragments(w[u][f][0], w[u][f][1], upper);
  #pragma unroll
        for (int b = 0; b < MB; b++) as_fragments(x[u][b][0], x[u][b][1], upper);
  #pragma unroll
        for (int h = 0; h < 2; h++)
  #pragma unroll
          for (int f = 0; f < NF; f++)
  #pragma unroll
            for (int b = 0; b < MB; b++)
              acc[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][f][h], x[u][b][h], acc[f][b], 0, 0, 0);
      }
    };
    // Groups of U steps are dealt over the wavefronts in turn - together they walk 128 U WAVES contiguous bytes of each row - then
    // single ones.  (No condition inside a group: under one, a step's loads sink to where it uses them.)
    typedef std::integral_constant<int, U> group;
    typedef std::integral_constant<int, 1> single;
    int s = wave * U;
    for (; s + U <= full; s += WAVES * U) steps(group(), std::false_type(), (int64_t)s * 64, 0);
    for (s = full / U * U + WAVES - 1 - wave; s < full; s += WAVES) steps(single(), std::false_type(), (int64_t)s * 64, 0);
    if ((p.K & 63) != 0 && wave == WAVES / 2 - 1)
      // what is left: the last 64 indices, without those of them that whole steps have counted
      steps(single(), std::true_type(), p.K - 64, 64 - (int)(p.K & 63));
  } else {
    const bf16_t* wp[NF];
    const bf16_t* xp[MB];
#pragma unroll
    for (int f = 0; f < NF; f++) {
      int n = n0 + (f % NB) * 16 + l16;
      n = n < p.N ? n : p.N - 1;
      wp[f] = (f < NB ? p.W : p.W2) + (int64_t)n * p.K + g * 8;
    }
#pragma unroll
    for (int b = 0; b < MB; b++) {
      int m = m0 + b * 16 + l16;
      m = m < p.M ? m : p.M - 1;
      xp[b] = p.X + (int64_t)m * p.K + g * 8;
    }
    const int full = (int)(p.K >> 5);                // whole steps of 32
    // groups of U steps are dealt over the wavefronts in turn: together they walk 64 U WAVES contiguous bytes of each row
    for (int s = wave * U; s < full; s += WAVES * U) {
      bf16x8 w[U][NF], x[U][MB];
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int64_t k = (int64_t)(s + u < full ? s + u : full - 1) * 32;   // past the end: the last step again, unused
#pragma unroll
        for (int f = 0; f < NF; f++) w[u][f] = load8<AL>(wp[f] + k);
#pragma unroll
        for (int b = 0; b < MB; b++) x[u][b] = load8<AL>(xp[b] + k);
      }
#pragma unroll
      for (int u = 0; u < U; u++)
        if (s + u < full) {                          // wave-uniform
#pragma unroll
          for (int f = 0; f < NF; f++)
#pragma unroll
            for (int b = 0; b < MB; b++) acc[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][f], x[u][b], acc[f][b], 0, 0, 0);
        }
    }
    if ((p.K & 31) != 0 && wave == WAVES - 1) {      // the last, partial step: element by element, zeros past the end
      const int64_t k = (int64_t)full * 32;
      bf16x8 w[NF], x[MB];
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const bool in = k + g * 8 + e < p.K;
#pragma unroll
        for (int f = 0; f < NF; f++) w[f][e] = in ? wp[f][k + e] : (bf16_t)0.0f;
#pragma unroll
        for (int b = 0; b < MB; b++) x[b][e] = in ? xp[b][k + e] : (bf16_t)0.0f;
      }
#pragma unroll
      for (int f = 0; f < NF; f++)
#pragma unroll
        for (int b = 0; b < MB; b++) acc[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[f], x[b], acc[f][b], 0, 0, 0);
    }
  }

  // pairwise over the wavefronts: the upper half hands its sums to the lower half until one is left
#pragma unroll
  for (int half = WAVES / 2; half >= 1; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int f = 0; f < NF; f++)
#pragma unroll
        for (int b = 0; b < MB; b++) red[wave - half][f * MB + b][lane] = acc[f][b];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
      for (int f = 0; f < NF; f++)
#pragma unroll
        for (int b = 0; b < MB; b++) {
          const f32x4 t = red[wave][f * MB + b][lane];
#pragma unroll
          for (int r = 0; r < 4; r++) acc[f][b][r] += t[r];
        }
    }
    if (half > 1) __syncthreads();                   // the slots are written again
  }
  if (wave != 0) return;

  // a lane holds columns n0 + 16 f + 4 g .. + 3 of row m0 + 16 b + l16
  const bool vec = (p.N & 3) == 0 && (p.ldo & 3) == 0;   // then a group of four columns exists whole or not at all
#pragma unroll
  for (int f = 0; f < NB; f++) {
    const int n = n0 + f * 16 + g * 4;
    if (n >= p.N) continue;
    float bias[4];
#pragma unroll
    for (int r = 0; r < 4; r++) bias[r] = (EPI != SK_GATE && p.bias != nullptr && n + r < p.N) ? p.bias[n + r] : 0.0f;
#pragma unroll
    for (int b = 0; b < MB; b++) {
      const int m = m0 + b * 16 + l16;
      if (m >= p.M) continue;
      const int64_t at = (int64_t)m * p.N + n, to = (int64_t)m * p.ldo + n;
      bf16x4 o;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        float v = acc[f][b][r];
        if (EPI == SK_GATE) {
          const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * v));
          v = v * sg * acc[NF - NB + f][b][r];
        } else {
          v += bias[r];
          if (EPI == SK_RELU) v = v > 0.0f ? v : 0.0f;
        }
        if (EPI == SK_MASK) o[r] = (v > 0.0f && n + r < p.N) ? p.aux[at + r] : (bf16_t)0.0f;
        else o[r] = (bf16_t)v;
      }
      if (vec) {
        *reinterpret_cast<bf16x4*>(p.out + to) = o;
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++)
          if (n + r < p.N) p.out[to + r] = o[r];
      }
    }
  }
}

// Reduction length from which whole lines are loaded (feed-forward block, us, 64-byte pieces / lines: 16 x 4096 x 11008 62.0 / 57.1,
// 1 x 4096 x 11008 52.8 / 48.5; at K = 1024 to 2000 equal within 2 %, below 1024 3 to 6 % slower: two steps of a wavefront or fewer).
// Four row blocks load X more than W.  Lines over pieces, whole calls, mean (and extremes) of 140 to 300 shapes each: gated, D 1024 to
// 4096 1.00 (0.88 - 1.07), beyond 0.97 (0.85 - 1.04); beside two column blocks, K 1024 to 2048 1.05 (up to 1.23), 2048 to 2900
// 1.02 (up to 1.15: inference 34 x 2176 x 9152 29.4 / 32.7 us), and beyond another kernel is picked.
constexpr int64_t kLinesFrom = 2048, kLinesFromGate4 = 4096;
template <int MB, int NB, int EPI, int WAVES, int U> void launch_skinny(SkinnyParams p, hipStream_t s) {
  p.mblocks = (p.M + 16 * MB - 1) / (16 * MB);
  const int strips = (p.N + 16 * NB - 1) / (16 * NB);
  const unsigned grid = (unsigned)((strips + 7) / 8 * 8) * (unsigned)p.mblocks;
  auto kern = p.K % 8 == 0 ? gemm_skinny_kernel<MB, NB, EPI, WAVES, U, true, false> : gemm_skinny_kernel<MB, NB, EPI, WAVES, U, false, false>;
  if constexpr (MB < 4 || NB == 1) {
    if (p.K >= (MB < 4 ? kLinesFrom : kLinesFromGate4))
      kern = p.K % 8 == 0 ? gemm_skinny_kernel<MB, NB, EPI, WAVES, 2, true, true> : gemm_skinny_kernel<MB, NB, EPI, WAVES, 2, false, true>;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * WAVES), 0, s, p);
}

// Tile and depth by the number of rows: the fewer there are, the more loads of W a wavefront can hold; from 33 rows on
// two column blocks share each load of X, and from 65 four row blocks each load of W where that still gives every compute
// unit a workgroup.
struct SkinnyTile { int mb, nb; };
SkinnyTile skinny_tile(int64_t M, int64_t N) {
  if (M <= 16) return {1, 1};
  if (M <= 32) return {2, 1};
  return {((N + 31) / 32) * ((M + 63) / 64) >= 256 ? 4 : 2, 2};
}
template <int EPI> void dispatch_skinny(const SkinnyParams& p, hipStream_t s) {
  const SkinnyTile t = skinny_tile(p.M, p.N);
  if (t.mb == 1) { launch_skinny<1, 1, EPI, 8, 8>(p, s); return; }
  if (t.nb == 1) { launch_skinny<2, 1, EPI, 8, 4>(p, s); return; }
  if constexpr (EPI == SK_GATE) {
    launch_skinny<4, 1, EPI, 8, 4>(p, s);
  } else {
    if (t.mb == 4) launch_skinny<4, 2, EPI, 8, 4>(p, s);
    else launch_skinny<2, 2, EPI, 8, 4>(p, s);
  }
}

}  // namespace

// Which kernel forms a forward product: the one with the lowest estimated time, the others charged 5 % (this one 10 %, with
// rows that start at any element 25 %) against the generic kernel, whose estimate is the steadier one.  This kernel rereads X for
// every 16 or 32 columns, so its time grows with its workgroups: per 256 of them a start and a price per element of K, which
// depends on the tile and on where rows start; above 4096 rows (2048 that start at any element) X no longer stays in the
// caches and the estimate no longer holds.  The tiled kernel's time is its own estimate, and the padded copies' where they are
// needed.  The prices are those of 64-byte loads and of the 32 x 32 x 16 tiles, which the present kernels beat by up to 15 and 8 %.  Inference,
// each kernel forced, the 128 x 128 tiles (offered after this) among them: on 3096 shapes (1 - 5000 rows, K to 8192, N to 16384) the kernel
// picked takes 1.015 times the fastest one's time on average, 1.07 at the 95th percentile, 1.6 at most; on 1476 of up to 300 rows and K from
// 2048 on 1.03, 1.18 and 2.1, nearly always this kernel where 128 x 128 tiles with a split reduction are faster, rows at any element above
// all (26 x 5323 x 664 40 / 19).  Measured with 64-byte loads, us, this kernel / generic: 4096 x 4096: 16 rows 10 / 87, 64 rows 20 / 88;
// 64 x 65536, 127 rows 36 / 16; 4097 x 65536: 31 rows 567 / 261, 127 rows 1169 / 293; this kernel / tiled: 4096 x 4096: 128 rows
// 29 / 31, 256 rows 48 / 35; 4096 x 1024: 384 rows 33 / 34, 1536 rows 72 / 41.
static int64_t skinny_rows(int64_t K) { return K % 8 == 0 ? 4096 : 2048; }
static double skinny_cost(int64_t M, int64_t K, int64_t N) {
  // start, per 256 workgroups, the same and 1000 elements of K, 1000 elements of K
  static const double price[4][2][4] = {
      {{2.6, 0.55, 1.2, 0.9}, {2.7, 0.70, 5.2, 2.0}},      // 1 x 1 blocks: K even, odd
      {{2.8, 0.43, 1.9, 1.6}, {3.0, 0.49, 8.4, 1.5}},      // 2 x 1
      {{3.5, 0.63, 1.0, 3.0}, {3.5, 0.43, 2.8, 9.7}},      // 2 x 2
      {{2.7, 1.8, 4.6, 1.2}, {3.1, 1.9, 14.0, 1.5}}};      // 4 x 2
  const SkinnyTile t = skinny_tile(M, N);
  const double* p = price[t.mb == 1 ? 0 : (t.nb == 1 ? 1 : (t.mb == 2 ? 2 : 3))][K % 2 == 0 ? 0 : 1];   // (4-byte addresses cost as much as 16-byte ones)
  const double wgs = (double)((N + 16 * t.nb - 1) / (16 * t.nb)) * (double)((M + 16 * t.mb - 1) / (16 * t.mb)) / 256.0;
  const double k = (double)K / 1000.0;
  return p[0] + (double)M / 2000.0 + wgs * (p[1] + p[2] * k) + p[3] * k;
}
Xwt pick_xwt(int64_t M, int64_t K, int64_t N, bool may_copy, bool may_pad, bool x_padded, double* cost_out) {
  Xwt best = Xwt::kGeneric;
  double cost = generic_xwt_cost(M, K, N);
  auto offer = [&](Xwt kernel, double c) { if (c < cost) { best = kernel; cost = c; } };
  const double skinny = M <= skinny_rows(K) ? skinny_cost(M, K, N) : 0.0;
  if (M <= skinny_rows(K)) offer(Xwt::kSkinny, skinny * (K % 8 == 0 ? 1.1 : 1.25));
  if (fast_f1_supported(M, K, N) && (may_copy || M % 256 == 0)) {
    // (a partial last row tile takes a copy of X's last rows, unless X has readable rows behind them)
    offer(Xwt::kTiled, 1.05 * (fast_xwt_cost(M, K, N, nullptr) + (M % 256 != 0 && !x_padded ? 4.0 : 1.0)));
  } else if (may_copy && may_pad && fast_padded_supported(M, K, N)) {
    const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K);
    const double copies = (double)(Np * Kp) * 2.0 + (fast_padded_stages_x(K) ? (double)(M * Kp) * 2.0 : 0.0);
    offer(Xwt::kPadded, 1.05 * (10.0 + fast_xwt_cost(M, K, N, nullptr) + copies / 3e6));
  }
  if (cost_out != nullptr) *cost_out = best == Xwt::kSkinny ? skinny : cost;
  return best;
}

// How the feed-forward block's gate and up products run, with what follows from it for the down product: the lowest estimated
// time of both.  The tiled gate kernel has a tile of 128 columns and no split; in padded mode it hands the activation on with a
// padded pitch, which the down product then takes in padded mode too.  This kernel's gate variant: about 10.5 us per 10^9
// products (row blocks of 64; the narrower ones count as 26 - 50 rows), a tenth more for rows at 4-byte addresses, three times that
// for rows that start at any element.  (Priced like the last, 330 shapes with even D that is no multiple of 8, 1 - 300 rows, lost 2 %
// to the faster of this kernel and the 128 x 128 tiles, up to 35 %: 21 x 3924 x 3698 26.7 us here, 42.6 there; now 0.1 %, below 5 %.)
// Measured, us, whole blocks: gate on this kernel / as two generic products: 16 x 4096 x 11008 64 / 478, 16 x 4097 x 11008 147 /
// 280, 66 x 4097 x 65536 2963 / 2120.
GatePlan pick_gate(int64_t M, int64_t D, int64_t H, bool can_pad) {
  GatePlan best = {Gate::kSeparate, Xwt::kGeneric, 0.0, 0.0};
  double down = 0.0;
  best.down = pick_xwt(M, H, D, true, can_pad && H % 128 == 0, /*x_padded=*/true, &down);
  const double mh = (double)M * (double)H;
  double cost = 2.0 * generic_xwt_cost(M, D, H) + 5.0 + mh * 6.0 / 4e6 + down;
  auto offer = [&](Gate gate, double c) { if (c < cost) { best.gate = gate; cost = c; } };
  const bool whole = D % 8 == 0, even = D % 2 == 0;
  const double rows = M <= 16 ? (whole ? 40.0 : 26.0) : (M <= 32 ? (whole ? 50.0 : 46.0) : (double)((M + 63) / 64 * 64));
  if (M <= skinny_rows(D))
    offer(Gate::kSkinny, 1.1 * (even && !whole ? 5.0 : 4.0) + 1.1 * (whole ? 10.5e-9 : (even ? 11.5e-9 : 34e-9)) * rows * (double)D * 2.0 * (double)H + down);
  const int64_t tiles = ((H + 127) / 128) * ((M + 255) / 256);
  const double tiled = (double)((tiles + 255) / 256) * ((double)D / 64 * 1.1 + 8.0);
  if (fast_gate_supported(M, D, H)) {
    offer(Gate::kTiled, 1.1 * tiled + down);
  } else if (can_pad) {
    const int64_t Hp = fast_gate_pad_h(H), Dq = fast_gate_pad_d(D);
    const double copies = (double)(Hp * Dq) * 4.0 + (double)(Hp * fast_pad_dim(D)) * 2.0 +
                          (fast_padded_stages_x(D) ? (double)(M * Dq) * 2.0 : 0.0);
    const double padded = 1.1 * (10.0 + copies / 3e6 + tiled + fast_xwt_cost(M, Hp, D, nullptr));
    if (padded < cost) { best.gate = Gate::kPadded; best.down = Xwt::kPadded; down = fast_xwt_cost(M, Hp, D, nullptr); cost = padded; }
  }
  best.gate_cost = cost - down;
  best.down_cost = down;
  return best;
}

// out[m][n] = f(sum_k X[m][k] W[n][k] + bias[n]): kind 0 plain (bias may be null), 1 max(., 0), 2 aux[m][n] where positive
void launch_skinny_xwt(int kind, int64_t M, int64_t K, int64_t N, const void* X, const void* W, const float* bias,
                       const void* aux, void* out, int64_t ldo, hipStream_t s) {
  SkinnyParams p = {};
  p.ldo = ldo;
  p.X = (const bf16_t*)X; p.W = (const bf16_t*)W; p.bias = bias; p.aux = (const bf16_t*)aux; p.out = (bf16_t*)out;
  p.K = K; p.M = (int)M; p.N = (int)N;
  if (kind == 1) dispatch_skinny<SK_RELU>(p, s);
  else if (kind == 2) dispatch_skinny<SK_MASK>(p, s);
  else dispatch_skinny<SK_STORE>(p, s);
}

// out[m][h] = SiLU(sum_d X[m][d] Wg[h][d]) * (sum_d X[m][d] Wu[h][d])
void launch_skinny_gate(int64_t M, int64_t D, int64_t H, const void* X, const void* Wg, const void* Wu, void* out, hipStream_t s) {
  SkinnyParams p = {};
  p.X = (const bf16_t*)X; p.W = (const bf16_t*)Wg; p.W2 = (const bf16_t*)Wu; p.out = (bf16_t*)out;
  p.K = D; p.M = (int)M; p.N = (int)H; p.ldo = H;
  dispatch_skinny<SK_GATE>(p, s);
}

}  // namespace fdl
