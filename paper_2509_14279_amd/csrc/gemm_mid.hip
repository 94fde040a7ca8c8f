// bf16 products of the sizes between a few rows and a chip full of 256 x 256 tiles (gfx950), any shape and alignment:
//
//     D[i][j] = sum_r P(i,r) * Q(j,r)      stored as C[j][i]   (operands and orientations as in gemm_bf16.hip)
//
//   forward  Z[m][n]  = sum_k X[m][k] W[n][k] + b[n]   P = W, Q = X, both r-contiguous
//   dX[m][k] = sum_n dZ[m][n] W[n][k]                  P = W (r-major), Q = dZ (r-contiguous)
//   dW[n][k] = sum_m dZ[m][n] X[m][k]                  P = X, Q = dZ, both r-major
//   H[m][h]  = SiLU(sum_d X[m][d] Wg[h][d]) * sum_d X[m][d] Wu[h][d]: the 128 rows of a P slice are 32 gate rows, the same 32 up
//   rows, the next 32 of each (a wave's blocks a = 0, 1 then hold both products of the same columns); 64 output columns per tile
//
// Bound: with one 128 x 128 tile per half of a compute unit, the operands' way from the L2 (a slice of 64 is 32 KB per tile for
// 2 MFLOP) and the latency of each slice's trip; the matrix cores are half idle.  What it has over the 256 x 256 tiles is up to
// four times as many of them - 3001 x 1537 has 84 of those on 256 compute units, 312 of these on 512 places - and no copies: rows
// are read as they lie.
// Measured, us, whole calls, before / with this kernel: forward product 2048 x 2048 x 2048 43 / 21 (800 TFLOP/s), 512 x 4096 x 4096
// 41 / 23, 3001 x 771 x 1537 39 / 23; both gradients of 1000 x 300 x 700 49 / 11, 16384 x 256 x 1024 56 / 28, 3001 x 771 x 1537
// 60 / 34; large ones stay with the other tiles: 8192 x 1024 x 4096 forward 63 to 76 here, gradients 120 to 140.
// Workgroup: 256 threads = 4 waves (2 x 2), block tile 128 x 128, wave tile 64 x 64 as 2 x 2 v_mfma_f32_32x32x16_bf16 blocks;
// slices of 64 through two LDS buffers (64 KB: two workgroups per compute unit cover each other's barriers), loads two slices
// ahead in registers, which any row alignment allows (direct loads to LDS want 4-byte addresses).
// LDS layouts as in gemm_bf16.hip, for 128 rows: r-contiguous [128 rows][8 chunks of 16 B], chunk c of row w in slot
// c ^ ((w >> 1) & 7); r-major [64 r-rows][16 chunks], chunk c of r-row w in slot c ^ ((w & 3) << 2).
#include "common.hip.h"
#include "internal.h"

#include <type_traits>

namespace fdl {
namespace {

enum { MID_STORE = 0, MID_RELU = 1, MID_MASK = 2, MID_PARTIAL = 3, MID_GATE = 4 };

constexpr int kMidTile = 128, kMidSlice = 64;
constexpr int kMidOperand = kMidTile * kMidSlice * 2;      // bytes of an operand's slice
constexpr int kMidLds = 2 * 2 * kMidOperand;

struct MidParams {
  const bf16_t* P; const bf16_t* Q;
  const bf16_t* P2;        // MID_GATE: the second P operand (same shape and pitch)
  int64_t ldp, ldq;
  bf16_t* C;               // [J][ldc]
  int64_t ldc;
  const float* bias;       // [I] or null
  const bf16_t* aux;       // [J][I] (MID_MASK)
  float* part;             // [split][J][I], pstride elements from part to part (MID_PARTIAL)
  int64_t pstride;
  int I, J, R;
  int rlen;                // reduction length of a part (a multiple of the slice)
  int split;
  int tiles_i, tiles_j;
};

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(2)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(1))) const char global_char;
typedef __attribute__((address_space(1))) const u32x4_u global_u32x4_u;
typedef __attribute__((ext_vector_type(4))) short short4_;
typedef __attribute__((address_space(3))) short4_ lds_short4;

// v, whose first element is element `skip` too early (8 and more: nothing of it is meant): the elements from there on, then zeros
__device__ __forceinline__ u32x4 drop_front(u32x4 v, int skip) {
  unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
  x = skip >= 8 ? 0 : x >> (16 * skip);
  return __builtin_bit_cast(u32x4, x);
}

// One operand's 128 x 64 slice; a thread moves four 16-byte chunks of it.  RM: r-major in memory.  TWO (r-contiguous): rows of two
// matrices in turn, 32 of each.
template <bool RM, bool TWO = false> struct MidSide {
  global_char* at;         // the slice fetched next (wave-uniform)
  global_char* at2;        // TWO: of the second matrix
  int64_t step;            // bytes from slice to slice
  uint32_t off[4];         // this thread's chunks
  uint32_t put;            // their place in LDS (4 KB apart)
  uint32_t get[4];         // the lane's fragments: RM by block of 32, else by sub-slice of 16

  // row of a slice that chunk q of this thread belongs to, in its matrix
  static __device__ __forceinline__ int row_of(int q, int tid) { return (tid >> 3) + 32 * (TWO ? q >> 1 : q); }
  // I rows of the operand (RM: columns) from i0 on; w: the wave's half
  __device__ __forceinline__ void init(const bf16_t* base, const bf16_t* base2, int64_t ld, int i0, int I, int64_t r0, int tid, int w) {
    const int lane = tid & 63;
    if (RM) {
      int c = (tid & 15) * 8;
      const int last = (I - 1 - i0) & ~7;                  // past the end: the last chunk again (its sums are not stored)
      c = c < last ? c : last;
#pragma unroll
      for (int q = 0; q < 4; q++) off[q] = (uint32_t)(((int64_t)((tid >> 4) + 16 * q) * ld + c) * 2);
      at = (global_char*)(base + r0 * ld + i0);
      step = (int64_t)kMidSlice * ld * 2;
      put = (uint32_t)((tid >> 4) * 256 + (((tid & 15) ^ (((tid >> 4) & 3) << 2)) << 4));
      const int g = lane >> 4, p = lane & 15;
#pragma unroll
      for (int a = 0; a < 2; a++) {
        const int ch = w * 8 + a * 4 + 2 * (g & 1) + ((p & 3) >> 1);
        get[a] = (uint32_t)((8 * (g >> 1) + (p >> 2)) * 256 + ((ch ^ ((p >> 2) << 2)) << 4) + (p & 1) * 8);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        int row = row_of(q, tid);
        row = row < I - i0 ? row : I - i0 - 1;
        off[q] = (uint32_t)(((int64_t)row * ld + (tid & 7) * 8) * 2);
      }
      at = (global_char*)(base + (int64_t)i0 * ld + r0);
      if (TWO) at2 = (global_char*)(base2 + (int64_t)i0 * ld + r0);
      step = kMidSlice * 2;
      put = (uint32_t)((tid >> 3) * 128 + (((tid & 7) ^ ((tid >> 4) & 7)) << 4));
      const int row = w * 64 + (lane & 31), t0 = (lane >> 5) ^ ((lane >> 1) & 7);
#pragma unroll
      for (int kk = 0; kk < 4; kk++) get[kk] = (uint32_t)(row * 128 + (((kk << 1) ^ t0) << 4));
    }
  }
  __device__ __forceinline__ u32x4 fetch(int q) const {
    uint32_t o = off[q];
    asm volatile("" : "+v"(o));      // (kept as 64-bit numbers the offsets take twice the registers)
    return *(global_u32x4_u*)((TWO && (q & 1) ? at2 : at) + o);
  }
  // The slice at r0, the last one, where it reaches past the reduction's end R or, RM, the end of the matrix: chunks that pass an
  // end are the last eight elements before it (I >= 8, R >= 8), which trim() moves to their place.
  __device__ __forceinline__ void aim_end(const bf16_t* base, const bf16_t* base2, int64_t ld, int i0, int I, int64_t r0, int64_t R, int tid) {
    if (RM) {
      const int c = i0 + (tid & 15) * 8, cc = c < I - 8 ? c : I - 8;
      const int rows = (int)(R - r0);
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int r = (tid >> 4) + 16 * q;
        off[q] = (uint32_t)(((int64_t)(r < rows ? r : rows - 1) * ld + cc) * 2);
      }
      at = (global_char*)(base + r0 * ld);
    } else {
      const int64_t r = r0 + (tid & 7) * 8, rc = r < R - 8 ? r : R - 8;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        int row = row_of(q, tid);
        row = row < I - i0 ? row : I - i0 - 1;
        off[q] = (uint32_t)(((int64_t)row * ld + rc) * 2);
      }
      at = (global_char*)(base + (int64_t)i0 * ld);
      if (TWO) at2 = (global_char*)(base2 + (int64_t)i0 * ld);
    }
  }
  // chunk q of that slice: zeros past the ends
  static __device__ __forceinline__ u32x4 trim(int q, u32x4 v, int i0, int I, int64_t r0, int64_t R, int tid) {
    if (RM) {
      const int c = i0 + (tid & 15) * 8;
      return drop_front(v, (tid >> 4) + 16 * q < R - r0 ? (c < I - 8 ? 0 : c - (I - 8)) : 8);
    }
    const int64_t r = r0 + (tid & 7) * 8;
    return drop_front(v, r < R - 8 ? 0 : (r < R ? (int)(r - (R - 8)) : 8));
  }
  __device__ __forceinline__ void stash(lds_char* lds, int q, u32x4 v) const { *(lds_u32x4*)(lds + put + q * 4096) = v; }
  __device__ __forceinline__ bf16x8 frag(const lds_char* lds, int a, int kk) const {
    if (RM) {
      const lds_char* p0 = lds + get[a] + kk * 4096;
      const short4_ lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p0);
      const short4_ hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p0 + 1024));
      typedef __attribute__((ext_vector_type(8))) short short8_;
      short8_ v;
      v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3]; v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
      return __builtin_bit_cast(bf16x8, v);
    } else {
      typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
      return *(const lds_bf16x8*)(lds + get[kk] + a * 4096);
    }
  }
};

inline int mid_units(const MidParams& p) { return (p.tiles_i * p.tiles_j + 7) / 8 * 8 * p.split; }

// unit `id` of a product (mid_units of them)
template <bool P_RM, bool Q_RM, int EPI>
__device__ __forceinline__ void mid_unit(const MidParams& p, const int id, char* smem) {
  lds_char* lds = (lds_char*)smem;
  // ids are dealt round-robin over 8 dies: a die takes neighbouring tiles, in bands of eight output-row tiles
  const int ntiles = p.tiles_i * p.tiles_j, per = (ntiles + 7) / 8;
  const int pt = id / (per * 8), slot = id - pt * per * 8, tile = (slot & 7) * per + (slot >> 3);
  if (tile >= ntiles) return;
  const int band = tile / (8 * p.tiles_i), rem = tile - band * 8 * p.tiles_i;
  const int band_h = p.tiles_j - band * 8 < 8 ? p.tiles_j - band * 8 : 8;
  constexpr bool kGate = EPI == MID_GATE;
  const int i0 = rem / band_h * (kGate ? kMidTile / 2 : kMidTile), j0 = (band * 8 + rem % band_h) * kMidTile;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wi = wave & 1, wj = wave >> 1;
  const int64_t r_begin = (int64_t)pt * p.rlen, r_end = r_begin + p.rlen < p.R ? r_begin + p.rlen : p.R;
  // Slices read with plain vectors: inside the reduction and, where a chunk of an r-major operand may pass its row's end (by
  // less than eight elements), not with the matrix's last row.
  const bool pass = (P_RM && (p.I + 7) / 8 * 8 > p.ldp) || (Q_RM && (p.J + 7) / 8 * 8 > p.ldq);
  const int64_t r_safe = pass && r_end == p.R ? p.R - 1 : r_end;
  const int full = r_safe > r_begin ? (int)((r_safe - r_begin) / kMidSlice) : 0;

  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[a][b][r] = 0.0f;
  typedef MidSide<P_RM, kGate> SP;
  typedef MidSide<Q_RM> SQ;
  SP sp; SQ sq;
  sp.init(p.P, p.P2, p.ldp, i0, p.I, r_begin, tid, wi);
  sq.init(p.Q, nullptr, p.ldq, j0, p.J, r_begin, tid, wj);
  const int total = (int)((r_end - r_begin + kMidSlice - 1) / kMidSlice);      // full, or one more: the end slice
  const int64_t r_last = r_begin + (int64_t)full * kMidSlice;
  if (total > 0) {
    // Issue order is pinned by hand (left to itself the compiler sinks the loads of a slice to where the next one waits for them
    // and reads fragments only when they are needed): behind each MFMA a fragment of the next sub-slice, a load of the slice
    // after next, or the next slice's way into LDS.  The last sub-slice's products come behind the barrier and the first
    // fragments of the next slice.
    u32x4 v[2][8];
    bf16x8 fp[2][2], fq[2][2];
    int ahead = 0;           // the slice that at and off name (past the last one they stay: it is fetched again, unused)
    auto advance = [&]() __attribute__((always_inline)) {
      ++ahead;
      const bool more = ahead < full;
      sp.at += more ? sp.step : 0;
      sq.at += more ? sq.step : 0;
      asm volatile("" : "+s"(sp.at), "+s"(sq.at));
      if constexpr (kGate) {
        sp.at2 += more ? sp.step : 0;
        asm volatile("" : "+s"(sp.at2));
      }
      if (ahead == full && full < total) {
        int t = tid;
        asm volatile("" : "+v"(t));    // (not to be worked out ahead of the loop)
        sp.aim_end(p.P, p.P2, p.ldp, i0, p.I, r_last, p.R, t);
        sq.aim_end(p.Q, nullptr, p.ldq, j0, p.J, r_last, p.R, t);
      }
    };
    auto load = [&](int q) __attribute__((always_inline)) { return q < 4 ? sp.fetch(q) : sq.fetch(q - 4); };
    auto put = [&](int buf, int q, u32x4 x) __attribute__((always_inline)) {
      lds_char* to = lds + buf * 2 * kMidOperand;
      if (q < 4) sp.stash(to, q, x); else sq.stash(to + kMidOperand, q - 4, x);
    };
    auto trim = [&](int q, u32x4 x) __attribute__((always_inline)) {
      int t = tid;
      asm volatile("" : "+v"(t));
      return q < 4 ? SP::trim(q, x, i0, p.I, r_last, p.R, t) : SQ::trim(q - 4, x, j0, p.J, r_last, p.R, t);
    };
    // fragment n of a sub-slice, in the order of their use: P0 Q0 Q1 P1
    auto read = [&](int buf, int kk, int n) __attribute__((always_inline)) {
      const lds_char* lp = lds + buf * 2 * kMidOperand;
      if (n == 0) fp[kk & 1][0] = sp.frag(lp, 0, kk);
      else if (n == 3) fp[kk & 1][1] = sp.frag(lp, 1, kk);
      else fq[kk & 1][n - 1] = sq.frag(lp + kMidOperand, n - 1, kk);
    };
    if (full == 0) {
      sp.aim_end(p.P, p.P2, p.ldp, i0, p.I, r_last, p.R, tid);
      sq.aim_end(p.Q, nullptr, p.ldq, j0, p.J, r_last, p.R, tid);
    }
#pragma unroll
    for (int q = 0; q < 8; q++) v[0][q] = load(q);
    advance();
#pragma unroll
    for (int q = 0; q < 8; q++) v[1][q] = load(q);
    advance();
#pragma unroll
    for (int q = 0; q < 8; q++) put(0, q, full == 0 ? trim(q, v[0][q]) : v[0][q]);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 4; n++) read(0, 0, n);
    // k: the LDS buffer; what: kMore - two more slices follow, kNext - one (the last), kLast - none
    enum { kMore, kNext, kLast };
    auto slice = [&](auto k_tag, auto what_tag) __attribute__((always_inline)) {
      constexpr int k = decltype(k_tag)::value, what = decltype(what_tag)::value;
      if (what == kNext && full < total) {
#pragma unroll
        for (int q = 0; q < 8; q++) v[k ^ 1][q] = trim(q, v[k ^ 1][q]);
      }
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        if (kk == 3 && what != kLast) { __syncthreads(); __builtin_amdgcn_sched_barrier(0); }
#pragma unroll
        for (int n = 0; n < 4; n++) {
          const int a = n >> 1, b = n & 1, t = kk * 4 + n;
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp[kk & 1][a], fq[kk & 1][b], acc[a][b], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (kk < 3) read(k, kk + 1, n);
          else if (what != kLast) read(k ^ 1, 0, n);
          __builtin_amdgcn_sched_barrier(0);
          if (what == kMore && t < 8) v[k][t] = load(t);
          if (what != kLast && t >= 4 && t < 12) put(k ^ 1, t - 4, v[k ^ 1][t - 4]);
          if (what == kMore && t == 8) advance();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    typedef std::integral_constant<int, 0> zero;
    typedef std::integral_constant<int, 1> one;
    typedef std::integral_constant<int, kMore> more;
    typedef std::integral_constant<int, kNext> next;
    typedef std::integral_constant<int, kLast> last;
    int left = total;
    for (; left >= 4; left -= 2) { slice(zero(), more()); slice(one(), more()); }
    if (left == 3) {
      slice(zero(), more()); slice(one(), next()); slice(zero(), last());
    } else if (left == 2) {
      slice(zero(), next()); slice(one(), last());
    } else {
      slice(zero(), last());
    }
  }

  // accumulator register r of block (a, b): i = a*32 + (r/4)*8 + (lane/32)*4 + r%4, j = b*32 + lane%32 of the wave tile
  const int half = lane >> 5, l32 = lane & 31;
  if (EPI == MID_PARTIAL) {
    typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
    float* out = p.part + (int64_t)pt * p.pstride;
#pragma unroll
    for (int b = 0; b < 2; b++) {
      const int j = j0 + wj * 64 + b * 32 + l32;
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const int i = i0 + wi * 64 + a * 32 + g * 8 + half * 4, left = p.I - i;
          if (j >= p.J) continue;
          float* dst = out + (int64_t)j * p.I + i;
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; e++) v[e] = acc[a][b][g * 4 + e];
          if (left >= 4) {
            *reinterpret_cast<f32x4_u*>(dst) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 4; e++)
              if (e < left) dst[e] = v[e];
          }
        }
    }
    return;
  }
  // The tile leaves through LDS as rows of 256 bytes (unit u of 8 bytes of row w in slot u ^ ((w & 15) << 1)).
  __syncthreads();
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  if constexpr (kGate) {
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int il = wi * 32 + g * 8 + half * 4;
#pragma unroll
      for (int b = 0; b < 2; b++) {
        const int row = wj * 64 + b * 32 + l32;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float z = acc[0][b][g * 4 + e], u = acc[1][b][g * 4 + e];
          v[e] = (bf16_t)(z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * z)) * u);
        }
        *(lds_bf16x4*)(lds + row * 256 + (((il >> 2) ^ ((row & 15) << 1)) << 3)) = v;
      }
    }
    __syncthreads();
    const int c8 = tid & 7, left = p.I - (i0 + c8 * 8);
#pragma unroll
    for (int it = 0; it < 4; it++) {
      const int row = it * 32 + (tid >> 3), j = j0 + row;
      if (j >= p.J || left <= 0) continue;
      const u32x4 v = *(const lds_u32x4*)(lds + row * 256 + ((c8 ^ (row & 15)) << 4));
      bf16_t* dst = p.C + (int64_t)j * p.ldc + i0 + c8 * 8;
      if (left >= 8) {
        *reinterpret_cast<u32x4_u*>(dst) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (e < left) reinterpret_cast<unsigned short*>(dst)[e] = (unsigned short)(v[e >> 1] >> ((e & 1) * 16));
      }
    }
    return;
  }
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int il = wi * 64 + a * 32 + g * 8 + half * 4;
      f32x4 bv = {0.0f, 0.0f, 0.0f, 0.0f};
      if (p.bias != nullptr) {
#pragma unroll
        for (int e = 0; e < 4; e++) bv[e] = p.bias[i0 + il + e < p.I ? i0 + il + e : p.I - 1];
      }
#pragma unroll
      for (int b = 0; b < 2; b++) {
        const int row = wj * 64 + b * 32 + l32;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float z = acc[a][b][g * 4 + e] + bv[e];
          v[e] = (bf16_t)(EPI == MID_RELU ? (z > 0.0f ? z : 0.0f) : z);
        }
        *(lds_bf16x4*)(lds + row * 256 + (((il >> 2) ^ ((row & 15) << 1)) << 3)) = v;
      }
    }
  __syncthreads();
  const int c8 = tid & 15, left = p.I - (i0 + c8 * 8);     // a lane's eight columns, and how many there are
#pragma unroll
  for (int it = 0; it < 8; it++) {
    const int row = it * 16 + (tid >> 4), j = j0 + row;
    if (j >= p.J || left <= 0) continue;
    u32x4 v = *(const lds_u32x4*)(lds + row * 256 + ((c8 ^ (row & 15)) << 4));
    if (EPI == MID_MASK) {
      // positive numbers, infinity among them (see EPI_MASK of the 256 x 256 kernel)
      const bf16_t* ap = p.aux + (int64_t)j * p.I + i0 + c8 * 8;
      u32x4 d = {0u, 0u, 0u, 0u};
      if (left >= 8) {
        d = *reinterpret_cast<const u32x4_u*>(ap);
      } else {
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (e < left) d[e >> 1] |= (uint32_t)reinterpret_cast<const unsigned short*>(ap)[e] << ((e & 1) * 16);
      }
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const uint32_t lo = ((v[e] & 0xffffu) - 1u) < 0x7f80u ? 0x0000ffffu : 0u;
        const uint32_t hi = ((v[e] >> 16) - 1u) < 0x7f80u ? 0xffff0000u : 0u;
        v[e] = d[e] & (lo | hi);
      }
    }
    bf16_t* dst = p.C + (int64_t)j * p.ldc + i0 + c8 * 8;
    if (left >= 8) {
      *reinterpret_cast<u32x4_u*>(dst) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 8; e++)
        if (e < left) reinterpret_cast<unsigned short*>(dst)[e] = (unsigned short)(v[e >> 1] >> ((e & 1) * 16));
    }
  }
}

template <int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_mid_kernel(MidParams p) {
  __shared__ __attribute__((aligned(1024))) char smem[kMidLds];
  mid_unit<false, false, EPI>(p, (int)blockIdx.x, smem);
}

// dX and dW side by side; the product with the longer units, whose last ones nothing follows to fill the chip, comes first.  Behind
// them, where no sums of split reductions need a launch of their own after this one, the column sums of the row pass
// (j.kinds ceil(N / 64) workgroups, as b2_kernel: a launch of 4 us for whatever it does).
template <int EPIA, int EPIB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_mid_pair_kernel(MidParams dx, MidParams dw, int first_units, int units, int dw_first, TailSums j) {
  __shared__ __attribute__((aligned(1024))) char smem[kMidLds];
  const int id = (int)blockIdx.x;
  if (EPIA == MID_STORE && EPIB == MID_STORE && id >= units) {
    const int cblocks = (int)((j.N + 63) / 64), which = (id - units) / cblocks;
    b2_columns<float, 4>(j.N, j.groups, j.kinds, j.colpart, (id - units) % cblocks, which,
                         which == 0 ? j.col_out[0] : (which == 1 ? j.col_out[1] : j.col_out[2]), reinterpret_cast<double (*)[64]>(smem));
    return;
  }
  const bool first = id < first_units;
  const int unit = first ? id : id - first_units;
  if (first == (dw_first != 0)) mid_unit<true, true, EPIB>(dw, unit, smem);
  else mid_unit<true, false, EPIA>(dx, unit, smem);
}

MidParams mid_params(const void* P, int64_t ldp, const void* Q, int64_t ldq, int64_t I, int64_t J, int64_t R, void* C, int64_t ldc,
                     int split, void* part) {
  MidParams p = {};
  p.P = (const bf16_t*)P; p.Q = (const bf16_t*)Q; p.ldp = ldp; p.ldq = ldq;
  p.C = (bf16_t*)C; p.ldc = ldc;
  p.part = (float*)part; p.pstride = partial_stride(I * J);
  p.I = (int)I; p.J = (int)J; p.R = (int)R;
  const int64_t slices = (R + kMidSlice - 1) / kMidSlice;
  p.split = split;
  p.rlen = (int)((slices + split - 1) / split * kMidSlice);
  p.tiles_i = (int)((I + kMidTile - 1) / kMidTile);
  p.tiles_j = (int)((J + kMidTile - 1) / kMidTile);
  return p;
}
int64_t mid_tiles(int64_t I, int64_t J) { return ((I + kMidTile - 1) / kMidTile) * ((J + kMidTile - 1) / kMidTile); }

}  // namespace

// the vectors of a matrix's end are its last eight elements; offsets inside a tile fit 32 bits
bool mid_supported(int64_t M, int64_t K, int64_t N) {
  const int64_t most = (int64_t)1 << 22;
  return M >= 1 && K >= 8 && N >= 8 && M <= most && K <= most && N <= most && mid_tiles(N, M) <= (1 << 20) &&
         mid_tiles(K, M) <= (1 << 20) && mid_tiles(K, N) <= (1 << 20);
}

// Estimated times, us.  256 compute units take the units of a launch in turn; two on one compute unit share it (a slice of both
// 0.87, of one alone 0.35 - 0.40, so that a second unit costs less than a third round).  Rows whose slices straddle cache lines cost
// more, those that start at odd elements more still; 4-byte addresses cost what 16-byte ones do.  The sums of a split reduction: a
// launch (forward; the gradients' are added by the launch that ends the pass anyway), their traffic, and a little per part.
// Fitted to 1300 shapes of 64 - 65536 rows, K to 4096, N to 16384 and up to 2^36 products, every split up to 8 (forward), 8 x 32
// (gradients): within 0.83 - 1.13 (forward), 0.80 - 1.19 (whole backward passes) of the measured time for 95 % of them.
double mid_xwt_cost(int64_t M, int64_t K, int64_t N, size_t room, int* split_out) {
  const int64_t tiles = mid_tiles(N, M), slices = (K + kMidSlice - 1) / kMidSlice;
  const double odd = K % 2 ? 1.27 : 1.0, lines = K % 64 ? 1.28 : 1.0, alone = K % 64 ? 1.16 : 1.0, mn = (double)M * (double)N / 1e6;
  const double load = (double)K * (double)(M + N) * 2.0 / 5e6;       // the operands, once, at 5 TB/s
  double best = 0.0;
  for (int split = 1; split <= 8; split++) {
    if (split > 1 && (slices < 2 * split || tiles * split > 1536 || fast_xwt_part_bytes(M, N, split) > room)) break;
    const int64_t held = (tiles * split + 255) / 256;
    const double len = (double)((slices + split - 1) / split) * odd;
    double cost = (double)(held / 2) * (len * lines * 0.865 - 0.9) + (double)(held % 2) * (len * alone * 0.35 + 0.2);
    if (cost < load) cost = load;
    cost += 6.0 + (K % 2 ? 0.7 : 0.0) + 0.53 * mn;
    if (split > 1) cost += 3.3 + 0.1 * split + 1.36 * split * mn;
    if (split == 1 || cost < best) { best = cost; *split_out = split; }
  }
  return best;
}
// How much lower this estimate has to be than another kernel's for a forward product to come here: 7 % for the estimates' spread;
// more where there are so few rows that the few-row kernel's own spread counts (1 - 16 rows, 211 shapes: with 7 % the kernel picked
// takes up to 1.46 times the other's time; 17 - 32 rows 1.3 times).
double mid_margin(int64_t M) { return M <= 16 ? 1.4 : (M <= 32 ? 1.2 : 1.07); }
double mid_grads_cost(int64_t M, int64_t K, int64_t N, size_t room, int* sa_out, int* sb_out) {
  const int64_t ta = mid_tiles(K, M), tb = mid_tiles(K, N), la = (N + kMidSlice - 1) / kMidSlice, lb = (M + kMidSlice - 1) / kMidSlice;
  const double odd = K % 2 ? 1.18 : 1.0, mk = (double)M * (double)K / 1e6, nk = (double)N * (double)K / 1e6;
  static const int parts[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
  double best = 0.0;
  *sa_out = *sb_out = 1;
  for (int sa : parts) {
    if (sa > 8 || (sa > 1 && (la < 4 * sa || ta * sa > 768))) break;
    const size_t na = sa > 1 ? (size_t)sa * partial_stride(M * K) * 4 : 0;
    if (na > room) break;
    for (int sb : parts) {
      if (sb > 1 && (lb < 4 * sb || tb * sb > 1024)) break;
      const size_t nb = sb > 1 ? (size_t)sb * partial_stride(N * K) * 4 : 0;
      if (na + nb > room) break;
      const double A = (double)((la + sa - 1) / sa), B = (double)((lb + sb - 1) / sb);
      const double units = (double)(ta * sa + tb * sb);
      const double rate = 0.39 * odd;
      double work = ((double)(ta * sa) * A + (double)(tb * sb) * B) / 256.0 * rate + units / 256.0 * 0.33;
      double one = (A > B ? A : B) * 0.4 * odd;                          // the longest unit, alone on its compute unit
      if (units > 256.0) {
        work += (A < B ? A : B) * rate * 1.1 * (units > 512.0 ? 1.0 : (units - 256.0) / 256.0);     // the last ones
        one *= 1.14;
      }
      double cost = (sa > 1 || sb > 1 ? 7.5 : 4.0) + (work > one ? work : one);     // (unsplit: no launch for sums follows)
      if (sa > 1) cost += sa * (mk + 0.11);
      if (sb > 1) cost += sb * (nk + 0.11);
      if ((sa == 1 && sb == 1) || cost < best) { best = cost; *sa_out = sa; *sb_out = sb; }
    }
  }
  // One to four columns of tiles (256 x 256 ones: one or two) read all of dZ each, and little else is read: of 2600 shapes those took 6 -
  // 10 us more than the above, by dZ's size up to 3 x 10^7 elements and no more beyond.
  if (K <= 512) {
    const double dz = 0.45 * (double)M * (double)N / 1e6;
    best += dz < 14.0 ? dz : 14.0;
  }
  return best;
}

void launch_mid_xwt(int kind, int64_t M, int64_t K, int64_t N, const void* X, const void* W, const float* bias, const void* aux,
                    void* out, int64_t ldo, int split, void* part, hipStream_t s) {
  MidParams p = mid_params(W, K, X, K, N, M, K, out, ldo, split, part);
  const dim3 grid((unsigned)mid_units(p));
  if (split > 1) {
    hipLaunchKernelGGL(gemm_mid_kernel<MID_PARTIAL>, grid, dim3(256), 0, s, p);
    launch_xwt_reduce(kind, split, part, p.pstride, M, N, bias, aux, out, ldo, s);
    return;
  }
  p.bias = bias; p.aux = (const bf16_t*)aux;
  auto kern = kind == 1 ? gemm_mid_kernel<MID_RELU> : (kind == 2 ? gemm_mid_kernel<MID_MASK> : gemm_mid_kernel<MID_STORE>);
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, p);
}

// out[m][h] = SiLU(sum_d X[m][d] Wg[h][d]) * (sum_d X[m][d] Wu[h][d]), out with pitch H
double mid_gate_cost(int64_t M, int64_t D, int64_t H) {
  int split;
  return mid_xwt_cost(M, D, 2 * H, 0, &split);
}
void launch_mid_gate(int64_t M, int64_t D, int64_t H, const void* X, const void* Wg, const void* Wu, void* out, hipStream_t s) {
  MidParams p = mid_params(Wg, D, X, D, H, M, D, out, H, 1, nullptr);
  p.P2 = (const bf16_t*)Wu;
  p.tiles_i = (int)((H + kMidTile / 2 - 1) / (kMidTile / 2));
  hipLaunchKernelGGL(gemm_mid_kernel<MID_GATE>, dim3((unsigned)mid_units(p)), dim3(256), 0, s, p);
}

void launch_mid_grads(const MidGrads& a, hipStream_t s) {
  const MidParams dx = mid_params(a.W, a.K, a.dZ, a.ldz, a.K, a.M, a.N, a.dX, a.K, a.sa, a.dxpart);
  const MidParams dw = mid_params(a.X, a.K, a.dZ, a.ldz, a.K, a.N, a.M, a.dW, a.K, a.sb, a.dwpart);
  const int nw = mid_units(dw), nx = mid_units(dx);
  auto kern = a.sa > 1 ? (a.sb > 1 ? gemm_mid_pair_kernel<MID_PARTIAL, MID_PARTIAL> : gemm_mid_pair_kernel<MID_PARTIAL, MID_STORE>)
                       : (a.sb > 1 ? gemm_mid_pair_kernel<MID_STORE, MID_PARTIAL> : gemm_mid_pair_kernel<MID_STORE, MID_STORE>);
  const bool dw_first = dw.rlen >= dx.rlen;
  const int cols = a.sa == 1 && a.sb == 1 ? a.cols.kinds * (int)((a.cols.N + 63) / 64) : 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)(nw + nx + cols)), dim3(256), 0, s, dx, dw, dw_first ? nw : nx, nw + nx, dw_first ? 1 : 0, a.cols);
}

}  // namespace fdl
