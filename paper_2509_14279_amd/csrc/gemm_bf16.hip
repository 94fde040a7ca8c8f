// bf16 MFMA GEMM for the three contractions of the fused dense-layer block (gfx950).
//
//     D[i][j] = sum_r P(i,r) * Q(j,r)      stored as C[j][i]   (C row-major, leading dimension I)
//
// P feeds the MFMA "A" side, Q the "B" side, so a lane ends up with 4 consecutive i (output columns) of one
// output row j in adjacent accumulator registers.
//
//   F1  Z[m][n]  = sum_k X[m][k] W[n][k] + b[n]   P = W (i = n, r-contiguous)   Q = X  (j = m, r-contiguous)
//       (also the forward product of the sibling operators: Linear+ReLU, its backward pass's recomputation of the
//        pre-activation with the activation mask applied to the upstream gradient, and the three products of the
//        gated feed-forward block)
//   B3  dX[m][k] = sum_n dZ[m][n] W[n][k]         P = W (i = k, r = n major)    Q = dZ (j = m, r-contiguous)
//   B4  dW[n][k] = sum_m dZ[m][n] X[m][k]         P = X (i = k, r = m major)    Q = dZ (j = n, r = m major)
//       (dZ is the library's own buffer and may be stored in 32 x 32 blocks, which suits both of its readers: Loader)
// (the linear layer's forward, grad-input and grad-weight products of the paper's linear tasks.)
//
// Workgroup: 256 threads = 4 waves (2 x 2), one per SIMD; block tile 256 x 256, wave tile 128 x 128 as 8 x 8
// v_mfma_f32_16x16x32_bf16 blocks (256 fp32 accumulators per lane, held in AGPRs).  Under matrix load the part's power limit
// sets its clock, and these MFMAs take less energy per product than v_mfma_f32_32x32x16_bf16, whose accumulators pass through
// the pipe once per 16 products instead of 32: a loop of nothing but MFMAs on normal random numbers 2010 against 1750 TFLOP/s on one
// machine, 2137 against 1866 on another (on zeros 2440 both).  Whole calls, us, 32 x 32 / 16 x 16 blocks: step 65536 x 2048 x 8192
// 5629 / 5440, 4096 x 4096 x 16384 1431 / 1365, 8192 x 1024 x 4096 266 / 258, Linear+ReLU 10000 x 1000 x 3000 291 / 276,
// feed-forward 16384 x 4096 x 11008 3319 / 3168.  The reduction runs in slices of
// BK through NS LDS stages (BK x NS = 64 x 2 or 32 x 4, 128 KB either way) filled by direct global->LDS loads
// (16 bytes per lane, no staging registers); the loads of slice kt+NS are issued as soon as slice kt's stage is
// released and stay in flight for NS-1 slice times while the MFMAs of the other stages run.  Workgroups are
// persistent (one per CU): the first slices of a workgroup's next tile are fetched during the last slices of its
// current one, and output tiles leave through a small LDS staging area as 256-byte row segments (short row
// segments cost write bandwidth: 8 or 16 bytes per lane straight from the registers measured 3 to 18 % slower).
// The number of slices per tile is a multiple of NS, so every slice's LDS stage is a compile-time constant.
//
// LDS tile layouts (XOR-swizzled by choosing which global chunk a lane fetches, since a direct load lands at
// base + lane*16).  The LDS of this part has 64 banks of 4 bytes; a 16-byte read serves the wavefront in four groups
// of 16 lanes - lanes {0-3, 12-15, 20-23, 24-27}, {4-11, 16-19, 28-31} and the same plus 32, measured with a pairwise
// conflict probe - and an 8-byte read in two groups of 32 consecutive lanes; a group completes in one cycle when
// its lanes touch 64 distinct banks.
//   r-contiguous operand: [256 rows][BK/8 chunks of 16 B]; BK = 64 (rows of 128 B, two rows per bank round): chunk c
//       of row w in slot c ^ ((w >> 1) & 7); BK = 32 (rows of 64 B, four rows per bank round): slot c ^ g((w >> 2) & 3) with
//       g = 0, 2, 3, 1; fragments are read with ds_read_b128 (lane l: 8 consecutive r, chunk l/16 of row l%16): a lane group has
//       rows 0-3 and 12-15 of one chunk and rows 4-11 of its neighbour, or the reverse, which then cover all 64 banks.
//   r-major operand:      [BK r-rows][32 chunks of 16 B]; chunk c of r-row w sits in slot c ^ ((w & 3) << 2) ^ ((w >> 2) & 2);
//       fragments are read with the transposing ds_read_b64_tr_b16 (4 consecutive r for the lane's column): the 32
//       lanes of a group read 32 bytes from each of 8 r-rows, which the swizzle spreads over the 256-byte bank round.
#include "common.hip.h"
#include "internal.h"

#include <type_traits>

namespace fdl {
namespace {

constexpr int kTile = 256;
// The launch plan (workspace sizes included) is host-only and must not depend on which device runs it, so the split
// of the dW reduction is planned for the part's 256 compute units; the launch itself asks the device.
constexpr int kPlanCUs = 256;
constexpr int kLdsStages = 128 * 1024;           // all pipeline stages together (2 x 64 KB or 4 x 32 KB)
constexpr int kLdsBytes = kLdsStages + 4 * 8192; // + 8 KB per wave, 4 for the output block rows and 0.5 for the bias = 160 KB

// Geometry of one pipeline configuration: reduction slices of BK, NS stages.
template <int BK> struct Geo {
  static constexpr int kSub = BK / 32;                    // MFMA sub-slices per slice
  static constexpr int kOperandBytes = kTile * BK * 2;    // one operand tile of one slice
  static constexpr int kStageBytes = 2 * kOperandBytes;   // P tile then Q tile
  static constexpr int kDpw = BK / 8;                     // direct-load instructions per operand, wave and slice
  static constexpr int kWaveBytes = kOperandBytes / 4;    // each wave fills a quarter of an operand tile
};

// EPI_STORE: C = acc.  EPI_BIAS: C = acc + bias.
// EPI_PARTIAL: fp32 partial sums of a split reduction.  EPI_RELU: C = max(acc + bias, 0).
// EPI_MASK: C = aux where acc + bias > 0, else 0 (aux [J][I]: the upstream gradient of a ReLU).
// EPI_GATE: two P operands (gate and up weights), C = SiLU(Q P^T) * (Q P2^T): see the kernel's p_origin.
enum { EPI_STORE = 0, EPI_BIAS = 2, EPI_PARTIAL = 3, EPI_RELU = 4, EPI_MASK = 5, EPI_GATE = 6 };

struct FastParams {
  const bf16_t* P; const bf16_t* Q;
  const bf16_t* P2;      // EPI_GATE: the second P operand (same shape and pitch as P)
  const bf16_t* Qtail;   // RAG: the Q rows of the last (partial) row tile as a padded 256-row copy, or null if Q
                         //      itself has readable rows up to the end of that tile
  int64_t ldp, ldq;
  bf16_t* C;             // [J][ldc]
  float* Cpart;          // [split][J][I] fp32, pstride elements from part to part (EPI_PARTIAL)
  const float* bias;     // [I]   (EPI_BIAS, EPI_RELU, EPI_MASK)
  const bf16_t* aux;     // [J][I] (EPI_MASK)
  int64_t ldc;           // row pitch of C (at least I)
  int64_t pstride;
  int I, J;              // J: valid output rows (RAG: any number >= 1; otherwise a multiple of 256)
  int tiles_i, tiles_j;
  int nkt;               // reduction slices per workgroup
  int split;
  int xcds;              // accelerator dies the workgroup ids are dealt over (1: no die-aware tile order)
  int pblocked;          // 1: P (r-contiguous, BK = 32: a copy of the weights, ldp columns) is stored in blocks of 32 x 32, see Loader
  int qblocked;          // 1: so is Q (the library's own dZ buffer, ldq columns)
  int cblocked;          // 1: the output C [J][I] is written in that blocked layout (EPI_MASK: the masked gradient;
                         //    EPI_GATE: the gated activation)
};

typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((ext_vector_type(4))) short short4_;
typedef __attribute__((address_space(3))) short4_ lds_short4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

// 16 bytes per lane, global -> LDS, no registers: lane l's data lands at (lds_base + LDS_OFF) + 16 l.
// voff: per-lane byte offset, sbase: wave-uniform global base, lds_base: wave-uniform LDS byte address.
// M0 carries the LDS address; one wait state separates the SALU write of M0 from the load that reads it.
template <int LDS_OFF>
__device__ __forceinline__ void dma16(uint32_t voff, const void* sbase, uint32_t lds_base) {
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(sbase), "s"(lds_base), "n"(LDS_OFF) : "memory", "m0", "scc");
}
// 4 bytes per lane: lane l's dword lands at (lds_base + LDS_OFF) + 4 l
template <int LDS_OFF>
__device__ __forceinline__ void dma4(uint32_t voff, const void* sbase, uint32_t lds_base) {
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :: "v"(voff), "s"(sbase), "s"(lds_base), "n"(LDS_OFF) : "memory", "m0", "scc");
}
// wait until at most N vector-memory operations of this wave are outstanding (loads complete in order)
template <int N> __device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// where chunks of 16 bytes sit in the LDS rows: chunk c in slot c ^ swizzle(row) (see the top of the file)
__device__ __forceinline__ int rm_swizzle(int w) { return ((w & 3) << 2) | ((w >> 2) & 2); }
__device__ __forceinline__ int rc32_swizzle(int w) { return (((w >> 2) ^ (w >> 3)) & 1) << 1 | ((w >> 3) & 1); }

template <bool RM, int BK> struct Loader {
  // voff[q]: per-lane byte offset of instruction q (constant over the reduction loop).  kDpw instructions per wave
  // fill this wave's quarter of the operand tile; the only per-slice scalar work is one base pointer.
  // Blocked operand (BK = 32 only): the matrix [rows][ld] is stored as [rows / 32][ld / 32] blocks of 32 x 32
  // elements, each block row-major and 2 KB long.  Either orientation then reads long runs: a 256-row slice of 32
  // reduction columns (r-contiguous use) is 8 whole blocks, a slice of 32 reduction rows by 256 columns (r-major use)
  // is 8 neighbouring blocks, 16 KB in one piece - where a row-major matrix gives the r-contiguous reader 256 runs of
  // 64 bytes, half a cache line each, whose other half it asks for again one slice later.  The 16-byte chunk a lane
  // fetches and the LDS slot it lands in are the same as for a row-major operand; only its address differs.
  static constexpr int kDpw = Geo<BK>::kDpw;
  uint32_t voff[kDpw];
  int blocked;
  __device__ __forceinline__ void init(int lane, int wave, int64_t ld, int blocked_operand = 0) {
    blocked = (BK == 32) ? blocked_operand : 0;
#pragma unroll
    for (int q = 0; q < kDpw; q++) {
      if (BK == 32 && blocked && RM) {
        // r-row 2q + h of this wave's 8 (all in one block row), chunk c: block c / 4, 16-byte piece c % 4 of its row
        const int h = lane >> 5, slot = lane & 31;
        const int c = slot ^ rm_swizzle(wave * (BK / 4) + 2 * q + h);
        voff[q] = (uint32_t)((c >> 2) * 2048 + (2 * q + h) * 64 + (c & 3) * 16);
      } else if (BK == 32 && blocked) {
        // row 16q + w of this wave's 64 (two block rows), piece slot ^ swizzle of its 64 bytes in the block
        const int w = lane >> 2, slot = lane & 3, rr = 16 * q + w;
        voff[q] = (uint32_t)((int64_t)(rr >> 5) * (ld >> 5) * 2048 + (rr & 31) * 64 + ((slot ^ rc32_swizzle(w)) * 16));
      } else if (RM) {
        // instruction q covers r-rows 2q, 2q+1 of this wave's BK/4; lane: r-row 2q + h, h = lane/32, slot lane%32
        const int h = lane >> 5, slot = lane & 31;
        const int c = slot ^ rm_swizzle(wave * (BK / 4) + 2 * q + h);
        voff[q] = (uint32_t)((int64_t)(2 * q + h) * ld * 2 + c * 16);
      } else if (BK == 64) {
        // instruction q covers rows 8q..8q+7 of this wave's 64; lane: row 8q + w, w = lane/8, slot lane%8
        const int w = lane >> 3, slot = lane & 7;
        voff[q] = (uint32_t)((int64_t)(8 * q + w) * ld * 2 + ((slot ^ ((4 * q + (w >> 1)) & 7)) * 16));
      } else {
        // BK = 32: instruction q covers rows 16q..16q+15 of this wave's 64; lane: row 16q + w, w = lane/4, slot lane%4
        const int w = lane >> 2, slot = lane & 3;
        voff[q] = (uint32_t)((int64_t)(16 * q + w) * ld * 2 + ((slot ^ rc32_swizzle(w)) * 16));
      }
    }
  }
  // first element this wave fetches of the slice that starts at `base` (block tile origin, first r of the slice)
  __device__ __forceinline__ const bf16_t* wave_base(const bf16_t* base, int64_t ld, int wave) const {
    if (BK == 32 && blocked) return RM ? base + wave * (BK / 4) * 32 : base + (int64_t)(wave * 2) * (ld >> 5) * 1024;
    return RM ? base + (int64_t)(wave * (BK / 4)) * ld : base + (int64_t)(wave * 64) * ld;
  }
  // wbase: wave_base(...) of the slice; wlds: LDS address of this wave's quarter of the operand tile
  template <int Q> __device__ __forceinline__ void issue1(const bf16_t* wbase, uint32_t wlds) const {
    dma16<Q * 1024>(voff[Q < kDpw ? Q : 0], wbase, wlds);
  }
  // q is a compile-time constant at every call site once the surrounding loop is unrolled
  __device__ __forceinline__ void issue_q(int q, const bf16_t* wbase, uint32_t wlds) const {
    switch (q) {
      case 0: issue1<0>(wbase, wlds); break;
      case 1: issue1<1>(wbase, wlds); break;
      case 2: issue1<2>(wbase, wlds); break;
      case 3: issue1<3>(wbase, wlds); break;
      case 4: if (kDpw > 4) issue1<4>(wbase, wlds); break;
      case 5: if (kDpw > 4) issue1<5>(wbase, wlds); break;
      case 6: if (kDpw > 4) issue1<6>(wbase, wlds); break;
      default: if (kDpw > 4) issue1<7>(wbase, wlds); break;
    }
  }
  __device__ __forceinline__ void issue(const bf16_t* wbase, uint32_t wlds) const {
#pragma unroll
    for (int q = 0; q < kDpw; q++) issue_q(q, wbase, wlds);
  }
};

template <bool RM, int BK> struct Frags {
  // LDS byte offsets of this lane's fragment reads inside an operand tile.
  //  r-contiguous: off[kk] for the sub-slices; block a adds a * 16 rows.
  //  r-major:      off[a] for the 8 blocks; sub-slice kk and half t add (kk*32 + 4t)*512.
  uint32_t off[8];
  __device__ __forceinline__ void init(int lane, int w /* wave coordinate along this operand */) {
    if (RM) {
      const int G = lane >> 4, p = lane & 15;
      const int r = 8 * G + (p >> 2);
#pragma unroll
      for (int a = 0; a < 8; a++) {
        const int c = w * 16 + a * 2 + ((p & 3) >> 1);
        off[a] = (uint32_t)(r * 512 + ((c ^ rm_swizzle(r)) * 16) + (p & 1) * 8);
      }
    } else {
      const int row = w * 128 + (lane & 15), c = lane >> 4;
      if (BK == 64) {
#pragma unroll
        for (int kk = 0; kk < 2; kk++) off[kk] = (uint32_t)(row * 128 + (((kk * 4 + c) ^ ((row >> 1) & 7)) << 4));
      } else {
        off[0] = (uint32_t)(row * 64 + ((c ^ rc32_swizzle(row)) << 4));
      }
    }
  }
  __device__ __forceinline__ bf16x8 load(const lds_char* tile, int a, int kk) const {
    if (RM) {
      const lds_char* p0 = tile + off[a] + (kk * 32) * 512;
      const short4_ lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p0);
      const short4_ hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p0 + 4 * 512));
      typedef __attribute__((ext_vector_type(8))) short short8_;
      short8_ v;
      v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3]; v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
      return __builtin_bit_cast(bf16x8, v);
    } else {
      typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
      return *(const lds_bf16x8*)(tile + off[kk] + a * (16 * BK * 2));
    }
  }
};

// Output tile of a logical tile index: bands of 8 output-row tiles, walked column-tile-major inside a band.
struct TileCoord { int i0, j0; };
__device__ __forceinline__ TileCoord tile_coord(int L, int tiles_i, int tiles_j) {
  const int band_tiles = 8 * tiles_i;
  const int band = L / band_tiles;
  const int rem = L - band * band_tiles;
  int band_h = tiles_j - band * 8;
  if (band_h > 8) band_h = 8;
  TileCoord c;
  c.i0 = (rem / band_h) * kTile;
  c.j0 = (band * 8 + rem % band_h) * kTile;
  return c;
}

// The MFMA with its accumulator in place, in AGPRs: left to choose, the register allocator moves accumulators about in straight
// code and parks some in scratch memory.  (Written as asm they are no MFMAs to the compiler, which would otherwise put wait states
// between one and a vector instruction that reads or has written its accumulator: the kernel does, and a host test looks at the built code.
// Its operands come from LDS, whose waits the compiler inserts for asm too.)
__device__ __forceinline__ void mfma_add(f32x4& acc, bf16x8 p, bf16x8 q) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(__builtin_bit_cast(u32x4, p)), "v"(__builtin_bit_cast(u32x4, q)));
}
__device__ __forceinline__ void mfma_start(f32x4& acc, bf16x8 p, bf16x8 q) {      // acc = p q
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(__builtin_bit_cast(u32x4, p)), "v"(__builtin_bit_cast(u32x4, q)));
}

// RAG: the number of output rows J is not a multiple of the tile (ragged batch dimension of F1 and B3, ragged N of
// B4).  The last row tile then reads its Q rows from a padded copy (or from a Q buffer that is itself padded), computes
// the surplus rows on whatever that padding holds - rows of a product are independent - and does not store them.
// CRAG (with RAG): the number of output columns I is any number, and so is the pitch of the output's rows (stores go to
// element-aligned addresses).  The host hands over a P operand that is readable up to the end of the last column tile (a
// zero-padded copy of the weights, or a matrix whose surplus columns are the start of its next row) and a bias padded
// likewise; the surplus columns are computed and not stored - EPI_MASK and EPI_GATE excepted, whose output, a buffer of the
// library with whole tiles of columns, gets zeros there.
// A reduction length that is not a whole number of pipeline rounds is the host's business as well: it rounds the
// length up and makes one operand zero over the surplus (the other only has to be readable and finite there).
// The body of the kernel: the persistent tile loop of workgroup `bid` of `nblk` on reduction part `part`.  It is a
// function of its own so that one launch can carry two contractions side by side (see gemm_bf16_pair_kernel).
template <bool P_RM, bool Q_RM, int EPI, int BK, int NS, bool RAG, bool CRAG = false>
__device__ __forceinline__ void gemm_tile_loop(const FastParams& p, char* smem, const int bid, const int nblk, const int part) {
  static_assert(!CRAG || RAG, "ragged columns come with the ragged-row checks");
  typedef Geo<BK> G;
  static_assert(NS * G::kStageBytes == kLdsStages, "stages must fill 128 KB");
  static_assert((NS == 2 || NS == 4) && ((NS * G::kSub) & 1) == 0, "2 or 4 stages, an even number of sub-slices in a round");
  lds_char* lds = (lds_char*)smem;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wi = wave & 1, wj = wave >> 1;

  // ---- persistent workgroups: one per CU, each walks several output tiles.  Workgroup ids are dealt round-robin
  // over the X accelerator dies (8 on this part), so die x owns the logical tiles [x T/X, (x+1) T/X) and its
  // workgroups take them in turn: the 32 workgroups resident on a die work on 32 consecutive logical tiles (4 column
  // tiles x 8 row tiles of one band) and share 4 P panels and 8 Q panels in that die's L2.  The host passes X > 1
  // only when both the tile count and the grid are multiples of it.
  const int ntiles = p.tiles_i * p.tiles_j;
  int L, Lstride, Lend;
  if (p.xcds > 1) {
    const int X = p.xcds;
    const int per_xcd = ntiles / X;
    const int xcd = bid % X, slot = bid / X;
    L = xcd * per_xcd + slot;
    Lstride = nblk / X;
    Lend = (xcd + 1) * per_xcd;
  } else {
    L = bid; Lstride = nblk; Lend = ntiles;
  }
  const int64_t r_begin = (int64_t)part * p.nkt * BK;

  // Per-lane offsets of the direct loads and of the fragment reads.  They are recomputed at the top of every tile
  // (from a copy of the lane id the compiler cannot see through) rather than kept across the epilogue, where the
  // register allocator would otherwise park them in scratch memory: a reload there has to wait for every output
  // store issued before it, because vector memory operations retire in order.
  Loader<P_RM, BK> lp; Loader<Q_RM, BK> lq;
  Frags<P_RM, BK> fp; Frags<Q_RM, BK> fq;
  auto init_offsets = [&]() {
    int lt = lane;
    asm volatile("" : "+v"(lt));
    lp.init(lt, wave, p.ldp, p.pblocked); lq.init(lt, wave, p.ldq, p.qblocked);
    fp.init(lt, wi); fq.init(lt, wj);
  };
  init_offsets();   // for the initial fill below; every tile recomputes them

  const bool pblk = BK == 32 && !P_RM && p.pblocked != 0;
  const int64_t pstep = P_RM ? (int64_t)BK * p.ldp : (pblk ? 1024 : BK);
  const bool qblk = BK == 32 && p.qblocked != 0;
  // (a slice step of an r-major operand is 32 rows = one block row either way: 32 ldq elements)
  const int64_t qstep = Q_RM ? (int64_t)BK * p.ldq : (qblk ? 1024 : BK);
  // first element this wave fetches of slice 0 of the tile at (i0, j0)
  // EPI_GATE: the 256 rows of a P tile are 64 gate rows, the same 64 up rows, the next 64 gate rows and their up rows
  // (rows of P and P2 from i0/2 on), one quarter per wave: a wave's accumulator blocks a = 0 .. 3 then hold the gate
  // product and a = 4 .. 7 the up product of the same 64 output columns, register for register, and the gated
  // activation needs no exchange between lanes.  The tile is 128 output columns wide.
  auto p_origin = [&](int i0) {
    if (pblk)    // block (i0 / 32, r_begin / 32)
      return lp.wave_base(p.P + ((int64_t)(i0 >> 5) * (p.ldp >> 5) + (r_begin >> 5)) * 1024, p.ldp, wave);
    if (EPI == EPI_GATE)
      return ((wave & 1) ? p.P2 : p.P) + (int64_t)((i0 >> 1) + (wave >> 1) * 64) * p.ldp + r_begin;
    return lp.wave_base(P_RM ? p.P + r_begin * p.ldp + i0 : p.P + (int64_t)i0 * p.ldp + r_begin, p.ldp, wave);
  };
  auto q_origin = [&](int j0) {
    if (RAG && !Q_RM && p.Qtail != nullptr && j0 == (p.tiles_j - 1) * kTile) return lq.wave_base(p.Qtail + r_begin, p.ldq, wave);
    if (qblk)   // block (j0 / 32, r_begin / 32), or (r_begin / 32, j0 / 32) for the r-major reader
      return lq.wave_base(Q_RM ? p.Q + ((r_begin >> 5) * (p.ldq >> 5) + (j0 >> 5)) * 1024
                               : p.Q + ((int64_t)(j0 >> 5) * (p.ldq >> 5) + (r_begin >> 5)) * 1024, p.ldq, wave);
    return lq.wave_base(Q_RM ? p.Q + r_begin * p.ldq + j0 : p.Q + (int64_t)j0 * p.ldq + r_begin, p.ldq, wave);
  };

  const int nkt = p.nkt;                                                  // >= NS
  const uint32_t wlds = lds0 + (uint32_t)wave * (uint32_t)G::kWaveBytes;  // this wave's quarter of an operand tile
  TileCoord tc = tile_coord(L, p.tiles_i, p.tiles_j);
  const bf16_t* pcur = p_origin(tc.i0);
  const bf16_t* qcur = q_origin(tc.j0);
#pragma unroll
  for (int st = 0; st < NS; st++) {
    lp.issue(pcur + st * pstep, wlds + st * G::kStageBytes);
    lq.issue(qcur + st * qstep, wlds + st * G::kStageBytes + G::kOperandBytes);
  }
  // the slice fetched last, as (addresses, index inside its tile)
  const bf16_t* pfetch = pcur + (NS - 1) * pstep;
  const bf16_t* qfetch = qcur + (NS - 1) * qstep;
  int fidx = NS - 1;
  constexpr bool kBias = EPI == EPI_BIAS || EPI == EPI_RELU || EPI == EPI_MASK;
  // The wave's 128 bias values go to the second half of its staging area by two direct loads at the top of the tile: no register and no
  // compiler-inserted wait is involved.
  const uint32_t wbias = (uint32_t)(kLdsStages + wave * 8192 + 4096);
  auto fetch_bias = [&](int i0) {
    int lb = lane;
    asm volatile("" : "+v"(lb));
    const float* bsrc = p.bias + i0 + wi * 128;
    dma4<0>((uint32_t)lb * 4u, bsrc, lds0 + wbias);
    dma4<256>((uint32_t)lb * 4u, bsrc + 64, lds0 + wbias);
  };
  wait_dma<0>();
  __syncthreads();

  // Fragments are double-buffered in registers: while the 64 MFMAs of a sub-slice run, the 16 fragment reads of the
  // next sub-slice (of 32) are issued between them.  The last sub-slice's MFMAs are issued after the barrier that
  // publishes the next stage, behind the first fragment reads of that stage, so the matrix pipe has work while
  // those reads are in flight.
  bf16x8 pf[2][8], qf[2][8];
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

  for (;;) {
    // slice 0 of this tile has landed in stage 0 (initial fill, or prefetched during the previous tile and
    // published by its last barrier): first fragments
    init_offsets();
#pragma unroll
    for (int n = 0; n < 8; n++) {
      if (n == 0) pf[0][0] = fp.load(lds, 0, 0);
      qf[0][n] = fq.load(lds + G::kOperandBytes, n, 0);
    }
#pragma unroll
    for (int a = 1; a < 8; a++) pf[0][a] = fp.load(lds, a, 0);

    // the tile after this one (its first NS slices are fetched during this tile's last NS slices); a workgroup
    // without a next tile fetches its own last slice again instead (never read)
    const int Ln = L + Lstride;
    const bool has_next = Ln < Lend;
    const TileCoord tn = tile_coord(has_next ? Ln : L, p.tiles_i, p.tiles_j);
    // where the fetch stream continues after this tile's last slice
    const bf16_t* pwrap = has_next ? p_origin(tn.i0) : p_origin(tc.i0) + (int64_t)(nkt - 1) * pstep;
    const bf16_t* qwrap = has_next ? q_origin(tn.j0) : q_origin(tc.j0) + (int64_t)(nkt - 1) * qstep;
    const int fwrap = has_next ? 0 : nkt - 1;

    f32x4 acc[8][8];                   // never cleared: the first MFMAs of a tile add to zero
    if (kBias) fetch_bias(tc.i0);      // (covered by the waits of this tile's slices, of which there are at least NS)

    // One slice; the LDS stage it lives in is a compile-time constant (the number of slices per tile is a multiple
    // of NS - checked on the host - so a tile's slice 0 is always in stage 0 and the slice loop is unrolled NS
    // times): every LDS address is then a per-lane register plus an immediate.
    auto slice = [&](auto stage_tag, auto first_tag) {
      constexpr bool kFirst = decltype(first_tag)::value;
      constexpr int cur = decltype(stage_tag)::value;
      constexpr int nxt = (cur + 1) & (NS - 1);
      // Slice kt+NS is fetched into this slice's own stage as soon as the barrier below has shown that every wave
      // holds its last fragments of slice kt in registers; those direct loads then have NS-1 slice times before
      // the barrier that publishes them.  (pfetch, qfetch, fidx) name the slice fetched last and are stepped in
      // the shadow of the last sub-slice's first MFMA: a handful of scalar instructions, where recomputing the
      // addresses from the slice index cost two dozen in front of every slice's first MFMA.
      const uint32_t own = wlds + (uint32_t)cur * G::kStageBytes;
      const lds_char* tp = lds + cur * G::kStageBytes;
      const lds_char* tq = tp + G::kOperandBytes;
      const lds_char* np_ = lds + nxt * G::kStageBytes;
      const lds_char* nq_ = np_ + G::kOperandBytes;
      // Issue order is pinned by hand (a scheduling barrier after every step): every third of the first 48 MFMAs of a sub-slice
      // is followed by a fragment read of the next sub-slice and, in the last sub-slice, every fourth or sixth by a direct load, so
      // neither the LDS reads nor the global loads keep the matrix pipe waiting for long.
#pragma unroll
      for (int kk = 0; kk < G::kSub; kk++) {
        const int use = (cur * G::kSub + kk) & 1, fill = use ^ 1;
        const bool lastsub = kk == G::kSub - 1;
        if (lastsub) {
          // Slice kt+1 must have landed; the direct loads of the NS-2 slices after it may stay in flight.  So may, in a tile's first
          // slices, whose successors were all fetched before them, the previous tile's stores (no fewer than counted: a lane's 16
          // bytes are an instruction each) and the bias: these all retire in order, and the stores' way to memory is long.
          constexpr int kStores = RAG ? 0 : (EPI == EPI_PARTIAL ? 64 : (EPI == EPI_GATE ? 16 : 32));
          constexpr int kBehind = kFirst && cur < NS - 1 ? kStores + (kBias ? 2 : 0) : 0, kFlying = (NS - 2) * 2 * G::kDpw + kBehind;
          wait_dma<kFlying < 63 ? kFlying : 63>();
          __syncthreads();
          __builtin_amdgcn_sched_barrier(0);
        }
        const lds_char* rp = lastsub ? np_ : tp;
        const lds_char* rq = lastsub ? nq_ : tq;
        const int rk = lastsub ? 0 : kk + 1;
#pragma unroll
        for (int t = 0; t < 64; t++) {
          const int a = t >> 3, b = t & 7;
          if (kFirst && cur == 0 && kk == 0) mfma_start(acc[a][b], pf[use][a], qf[use][b]);
          else mfma_add(acc[a][b], pf[use][a], qf[use][b]);
          __builtin_amdgcn_sched_barrier(0);
          // next slice of the fetch stream: the following one of this tile, else (pwrap, qwrap, fwrap) = slice 0
          // of the next tile or, without a next tile, this tile's last slice again, which is never read; spread
          // over three MFMA shadows
          if (lastsub && t == 0) {
            pfetch = fidx + 1 == nkt ? pwrap : pfetch + pstep;
            __builtin_amdgcn_sched_barrier(0);
          }
          if (lastsub && t == 2) {
            qfetch = fidx + 1 == nkt ? qwrap : qfetch + qstep;
            __builtin_amdgcn_sched_barrier(0);
          }
          if (lastsub && t == 4) {
            fidx = fidx + 1 == nkt ? fwrap : fidx + 1;
            __builtin_amdgcn_sched_barrier(0);
          }
          const bf16_t* const pn = pfetch;
          const bf16_t* const qn = qfetch;
          if (t % 3 == 0 && t < 48) {
            // read order: P0, Q0 .. Q7, P1 .. P7 (the order in which the next sub-slice consumes them)
            const int slot = t / 3;
            if (slot == 0) pf[fill][0] = fp.load(rp, 0, rk);
            else if (slot <= 8) qf[fill][slot - 1] = fq.load(rq, slot - 1, rk);
            else pf[fill][slot - 8] = fp.load(rp, slot - 8, rk);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (lastsub) {
            // The direct loads, as far apart as the sub-slice allows: bunched they fill the memory pipe's queue, and a wave that
            // waits to issue one issues no MFMA either (forward product 4096 x 4096 x 16384, 16 loads behind every second /
            // fourth MFMA 466 / 420 us).
            constexpr int kEvery = G::kDpw == 8 ? 4 : 6;
            if (t < 2 * G::kDpw * kEvery && t % kEvery == 2) {
              const int d = t / kEvery;
              if (d < G::kDpw) lp.issue_q(d, pn, own);
              else lq.issue_q(d - G::kDpw, qn, own + G::kOperandBytes);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
    };
    auto group = [&](auto first_tag) {
      slice(std::integral_constant<int, 0>(), first_tag);
      slice(std::integral_constant<int, 1>(), first_tag);
      if constexpr (NS == 4) {
        slice(std::integral_constant<int, 2>(), first_tag);
        slice(std::integral_constant<int, 3>(), first_tag);
      }
    };
    group(std::true_type());
    for (int g = NS; g < nkt; g += NS) group(std::false_type());
    // here: the next tile's slice 0 has landed in stage 0, its following slices are in flight

    // ---------------------------------------------------------------- epilogue of tile (tc.i0, tc.j0)
    // Accumulator register r of block (a, b): i = a*16 + (lane/16)*4 + r, j = b*16 + lane%16.  A lane's
    // four adjacent values are only 8 bytes of an output row, so bf16 tiles leave through LDS: each wave owns 4 KB
    // beyond the pipeline stages, writes one block row (16 output rows x 256 B) as [16 rows][32 units of 8 B] with
    // unit u of row w in slot u ^ (w << 1) (conflict-free both ways), reads it back 16 bytes per lane and
    // stores 256 contiguous bytes per row.
    // Every per-lane constant of the epilogue is derived here from a copy of the lane id the compiler cannot see
    // through: hoisted out of the tile loop they would be spilled around the main loop, and each reload in the
    // epilogue would wait for the output stores issued before it (vector memory operations retire in order).
    asm volatile("s_nop 15\n\ts_nop 15");      // (the last MFMAs' results)
#pragma unroll
    for (int a = 0; a < 8; a++)
#pragma unroll
      for (int b = 0; b < 8; b++) asm volatile("" : "+a"(acc[a][b]));
    int le = lane;
    asm volatile("" : "+v"(le));
    const int i0 = tc.i0, j0 = tc.j0;
    const uint32_t wtile = lds0 + (uint32_t)(kLdsStages + wave * 8192);
    // e_m, e_rq: column group and row of four (accumulators: row and column group)
    const int e_m = le & 15, e_rq = le >> 4;
    uint32_t woff[8];                            // LDS address of the lane's 8-byte unit a in row lane%16
#pragma unroll
    for (int a = 0; a < 8; a++) {
      woff[a] = wtile + (uint32_t)(e_m * 256 + (((a * 4 + e_rq) ^ (e_m << 1)) << 3));
      asm volatile("" : "+v"(woff[a]));
    }
    // read side: rows it*4 + lane/16 of the block row, 16-byte chunk lane%16 (slot chunk ^ row)
    uint32_t roff[4];
#pragma unroll
    for (int it = 0; it < 4; it++) {
      // (EPI_GATE: 16-byte chunk lane%8 of rows it*8 + lane/8)
      if (EPI == EPI_GATE) roff[it] = wtile + (uint32_t)((it * 8 + (le >> 3)) * 256 + (((le & 7) ^ (it * 8 + (le >> 3))) << 4));
      else roff[it] = wtile + (uint32_t)((it * 4 + e_rq) * 256 + ((e_m ^ (it * 4 + e_rq)) << 4));
      asm volatile("" : "+v"(roff[it]));
    }
    // Block row b: stage() rounds it into the staging area, collect() reads it back as rows, store_rows() sends those out.  One
    // row's stores are issued behind the conversions of the next, which cover the trip through LDS (a wave's LDS operations stay in
    // order, so one area serves them all): the tile end of the
    // forward product 65536 x 2048 x 8192 was 10 % of its 1630 us, 26 of which this and the accumulators kept in place give back.
    constexpr int kCollect = EPI == EPI_GATE ? 2 : 4;
    u32x4 rows[2][4];
    auto collect = [&](int b) {
#pragma unroll
      for (int it = 0; it < kCollect; it++) rows[b & 1][it] = *(const lds_u32x4*)(uintptr_t)roff[it];
    };
    const uint32_t svoff = (uint32_t)(e_rq * (int)p.ldc + e_m * 8) * 2u;   // byte offset of the lane inside 4 output rows
    typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(2)));
    // EPI_MASK: the upstream gradient of a block row, fetched while the two before it leave.  (Fetched where it is used, a tile
    // made many trips to memory in a row.  Linear+ReLU backward, us, that / so: 10000 x 1000 x 3000 248 / 217, 20000 x 512 x 2048
    // 224 / 184, 16384 x 1000 x 3001 385 / 324, 65536 x 2048 x 8192 5388 / 5020.)  Rows past the end are the last
    // one again; a lane whose eight columns pass the end takes the last eight, moved to their place, with zeros behind.
    u32x4 aux[3][4];
    auto fetch_aux = [&](int b) {
      if (EPI != EPI_MASK) return;
      const int left = CRAG ? p.I - (i0 + wi * 128 + e_m * 8) : 8, early = left >= 8 ? 0 : 8 - left;
#pragma unroll
      for (int it = 0; it < 4; it++) {
        int row = j0 + wj * 128 + b * 16 + it * 4 + e_rq;
        if (RAG) row = row < p.J ? row : p.J - 1;
        const bf16_t* ap = p.aux + (int64_t)row * p.I + (i0 + wi * 128 + e_m * 8 - early);
        if (CRAG) aux[b % 3][it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(ap));
        else aux[b % 3][it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ap));
      }
    };
    auto place_aux = [&](int b) {
      if (EPI != EPI_MASK || !CRAG) return;
      const int left = p.I - (i0 + wi * 128 + e_m * 8);
      if (left >= 8) return;
#pragma unroll
      for (int it = 0; it < 4; it++) {
        const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, aux[b % 3][it]);
        aux[b % 3][it] = __builtin_bit_cast(u32x4, left <= 0 ? (unsigned __int128)0 : x >> (16 * (8 - left)));
      }
    };
    auto store_rows = [&](int b) {
      place_aux(b);
      // wave-uniform base of row it*4 of the block row; the lane adds (lane/16) rows and 16 (lane%16) bytes
      char* cbase = reinterpret_cast<char*>(p.C + (int64_t)(j0 + wj * 128 + b * 16) * p.ldc + i0 + wi * 128);
#pragma unroll
      for (int it = 0; it < 4; it++) {
        const u32x4 v = rows[b & 1][it];
        u32x4* dst = reinterpret_cast<u32x4*>(cbase + (int64_t)(it * 4) * p.ldc * 2 + svoff);
        if (EPI == EPI_MASK && p.cblocked) {
          // row R0 + lane/16 (R0 a multiple of 4, so the four rows share a block row), columns col .. col + 7:
          // four rows x 64 bytes of each of the four blocks = 256 contiguous bytes per block
          const int64_t R0 = j0 + wj * 128 + b * 16 + it * 4;
          const int col = i0 + wi * 128 + e_m * 8;
          dst = reinterpret_cast<u32x4*>(p.C + (((R0 >> 5) * (p.I >> 5) + (col >> 5)) << 10) + (((R0 & 31) + e_rq) << 5) + (col & 31));
        }
        if (RAG && j0 + wj * 128 + b * 16 + it * 4 + e_rq >= p.J) continue;   // a row past the end
        const int cleft = CRAG ? p.I - (i0 + wi * 128 + e_m * 8) : 8;          // columns from this lane's first to the end
        if (CRAG && EPI != EPI_MASK) {
          if (cleft >= 8) {
            if (kBias) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_u*>(dst));
            else *reinterpret_cast<u32x4_u*>(dst) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 8; e++)
              if (e < cleft) reinterpret_cast<unsigned short*>(dst)[e] = (unsigned short)(v[e >> 1] >> ((e & 1) * 16));
          }
          continue;
        }
        if (EPI == EPI_MASK) {
          // v: 8 pre-activations as bf16.  The upstream gradient passes where the pre-activation is positive (bits
          // 0x0001 .. 0x7f80: sign clear, magnitude non-zero, up to infinity) and is zero elsewhere, NaN included.
          const u32x4 d = aux[b % 3][it];
          u32x4 g;
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const uint32_t lo = ((v[e] & 0xffffu) - 1u) < 0x7f80u ? 0x0000ffffu : 0u;
            const uint32_t hi = ((v[e] >> 16) - 1u) < 0x7f80u ? 0xffff0000u : 0u;
            g[e] = d[e] & (lo | hi);
          }
          *dst = g;
          continue;
        }
        // the forward output (Zsave, far larger than the caches) is streamed past them so that it does not evict
        // the operand panels the XCD's workgroups share; the smaller gradient outputs gain nothing from that
        if (kBias && EPI != EPI_MASK) __builtin_nontemporal_store(v, dst);
        else *dst = v;
      }
    };
    if (EPI == EPI_GATE) {
      // H = SiLU(gate) * up for this wave's 64 columns x 128 rows, one block row of 16 rows at a time through the
      // staging area (units 0..15 of each 256-byte staging row), stored as 128-byte row segments
      const int h0 = (i0 >> 1) + wi * 64;
      const int g_m = le & 7, g_rq = le >> 3;
      auto stage = [&](int b) {
#pragma unroll
        for (int a = 0; a < 4; a++) {
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const float z = acc[a][b][e], u = acc[a + 4][b][e];
            const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * z));
            v[e] = (bf16_t)(z * sg * u);
          }
          *(lds_bf16x4*)(uintptr_t)woff[a] = v;
        }
      };
      stage(0);
      collect(0);
#pragma unroll
      for (int b = 0; b < 8; b++) {
        __builtin_amdgcn_sched_barrier(0);
        if (b < 7) stage(b + 1);
        __builtin_amdgcn_sched_barrier(0);
        char* cbase = reinterpret_cast<char*>(p.C + (int64_t)(j0 + wj * 128 + b * 16) * p.ldc + h0);
#pragma unroll
        for (int it = 0; it < 2; it++) {
          const int row = it * 8 + g_rq;
          u32x4 v = rows[b & 1][it];
          if (RAG && j0 + wj * 128 + b * 16 + row >= p.J) continue;   // a row past the end
          if (CRAG && h0 + g_m * 8 + 8 > p.I) {
            // the surplus columns of a padded width are zeros (their sums are too, but not where X holds an infinity)
#pragma unroll
            for (int e = 0; e < 8; e++)
              if (h0 + g_m * 8 + e >= p.I) v[e >> 1] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;
          }
          if (p.cblocked) {
            // blocked output (the down projection reads it best that way): row R of the matrix, columns col .. col + 7
            const int64_t R = j0 + wj * 128 + b * 16 + row;
            const int col = h0 + g_m * 8;
            *reinterpret_cast<u32x4*>(p.C + (((R >> 5) * (p.I >> 5) + (col >> 5)) << 10) + ((R & 31) << 5) + (col & 31)) = v;
            continue;
          }
          *reinterpret_cast<u32x4*>(cbase + ((int64_t)row * p.ldc + g_m * 8) * 2) = v;
        }
        __builtin_amdgcn_sched_barrier(0);
        if (b < 7) collect(b + 1);
      }
    } else if (EPI == EPI_PARTIAL) {
      // fp32 partial sums of this reduction part, straight from the registers (wave-uniform base + lane offset)
      float* out = p.Cpart + (int64_t)part * p.pstride;
      typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
      const uint32_t pvoff = (uint32_t)(e_m * p.I + e_rq * 4) * 4u;
#pragma unroll
      for (int b = 0; b < 8; b++) {
        char* obase = reinterpret_cast<char*>(out + (int64_t)(j0 + wj * 128 + b * 16) * p.I + i0 + wi * 128);
#pragma unroll
        for (int a = 0; a < 8; a++) {
          if (RAG && j0 + wj * 128 + b * 16 + e_m >= p.J) continue;                     // a row past the end
          float* dst = reinterpret_cast<float*>(obase + a * 64 + pvoff);
          const int cleft = CRAG ? p.I - (i0 + wi * 128 + a * 16 + e_rq * 4) : 4;       // columns to the end
          if (CRAG && cleft < 4) {
#pragma unroll
            for (int e = 0; e < 4; e++)
              if (e < cleft) dst[e] = acc[a][b][e];
          } else if (CRAG) {
            *reinterpret_cast<f32x4_u*>(dst) = acc[a][b];
          } else {
            *reinterpret_cast<f32x4*>(dst) = acc[a][b];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      // rounded to bf16 and stored (the row statistics are taken by the normalisation kernel).  The bias is added to the finished sum: one
      // rounding, where a sum that starts from it has one at the bias's size for every 32 products (values of Z that are not the nearest
      // bf16 to the exact one, 4096 x 8192 x 4096, |b| 1000 times the products: 1.1e-4, so 3e-7).  It takes 256 additions per lane and tile.
      f32x4 bias[8];                   // of columns a * 16 + e_rq * 4 + e
      if (kBias)
#pragma unroll
        for (int a = 0; a < 8; a++) bias[a] = *(const lds_f32x4*)(lds + wbias + e_rq * 16 + a * 64);
      auto stage = [&](int b) {
#pragma unroll
        for (int a = 0; a < 8; a++) {
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const float z = kBias ? acc[a][b][e] + bias[a][e] : acc[a][b][e];
            v[e] = (bf16_t)(EPI == EPI_RELU ? __builtin_fmaxf(z, 0.0f) : z);
          }
          *(lds_bf16x4*)(uintptr_t)woff[a] = v;
        }
      };
      fetch_aux(0);
      fetch_aux(1);
      stage(0);
      collect(0);
#pragma unroll
      for (int b = 0; b < 8; b++) {
        __builtin_amdgcn_sched_barrier(0);   // one block row at a time: keeps the accumulator copies in few registers
        if (b < 6) fetch_aux(b + 2);
        if (b < 7) stage(b + 1);
        __builtin_amdgcn_sched_barrier(0);
        store_rows(b);
        __builtin_amdgcn_sched_barrier(0);
        if (b < 7) collect(b + 1);
      }
    }

    if (!has_next) break;
    L = Ln; tc = tn;
  }
  wait_dma<0>();   // the re-fetches issued during the last tile must land before the workgroup may retire
}

template <bool P_RM, bool Q_RM, int EPI, int BK, int NS, bool RAG, bool CRAG = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_bf16_kernel(FastParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_tile_loop<P_RM, Q_RM, EPI, BK, NS, RAG, CRAG>(p, smem, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y);
}

// Two contractions in one launch: the dX product on the first na * (parts of its reduction) workgroups and the dW
// product on the rest (nb workgroups per part of its reduction); a split reduction writes fp32 partial sums.  For
// outputs so small that neither contraction has a tile for every compute unit - a dX with few column tiles, a small
// dW - the two together still fill the chip, where two launches in a row would each leave part of it idle.
template <int BK, int NS, int EPIA, int EPIB, bool RAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_bf16_pair_kernel(FastParams pa, FastParams pb, int na, int nb) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int id = (int)blockIdx.x, a_all = na * pa.split;
  if (id < a_all) {
    gemm_tile_loop<true, false, EPIA, BK, NS, RAG, RAG>(pa, smem, id % na, na, id / na);
  } else {
    const int t = id - a_all;
    gemm_tile_loop<true, true, EPIB, BK, NS, RAG, RAG>(pb, smem, t % nb, nb, t / nb);
  }
}

// src [rows][cols] in blocks of 32 x 32 (see Loader; rows multiples of 32, cols of 64): a workgroup moves two neighbouring blocks,
// 128 bytes of each of 32 rows.
__global__ __launch_bounds__(256) void block32_kernel(const bf16_t* __restrict__ src, int64_t cols, bf16_t* __restrict__ dst) {
  const int row = threadIdx.x >> 3, chunk = threadIdx.x & 7;
  const int64_t b = blockIdx.y, c0 = (int64_t)blockIdx.x * 64;
  const u32x4 v = *reinterpret_cast<const u32x4*>(src + (b * 32 + row) * cols + c0 + chunk * 8);
  const int64_t to = b * (cols >> 5) + (c0 >> 5) + (chunk >> 2);
  *reinterpret_cast<u32x4*>(dst + to * 1024 + row * 32 + (chunk & 3) * 8) = v;
}

// Zero-padded copies, several in one launch (they are small dependent launches otherwise, a few microseconds each):
// job k: dst [rows_out][cols_out] = src [rows][cols] with zeros around it (src null: all zeros), cols_out a multiple of 8,
// src rows `ld` elements apart at any element; then the fp32 vector vdst [vn_out] = vsrc [vn] and zeros.
__global__ __launch_bounds__(256) void stage_kernel(StageJobs j) {
  typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(2)));
  int id = (int)blockIdx.x;
  for (int k = 0; k < j.count; k++) {
    const StageJob& q = j.job[k];
    if (id >= q.blocks) { id -= q.blocks; continue; }
    const int64_t vpr = q.cols_out / 8;                      // vectors per row
    const int per = vpr < 256 ? (int)(256 / vpr) : 1;        // rows a workgroup copies at a time
    const int tr = vpr < 256 ? (int)threadIdx.x / (int)vpr : 0;
    const int64_t tc = vpr < 256 ? (int)threadIdx.x % (int)vpr : threadIdx.x;
    if (tr >= per) return;
    const unsigned short* src = static_cast<const unsigned short*>(q.src);
    unsigned short* dst = static_cast<unsigned short*>(q.dst);
    for (int64_t r = (int64_t)id * per + tr; r < q.rows_out; r += (int64_t)q.blocks * per)
      for (int64_t v = tc; v < vpr; v += 256) {
        const int64_t c = v * 8;
        u32x4 x = {0u, 0u, 0u, 0u};
        if (src != nullptr && r < q.rows) {
          const unsigned short* s = src + r * q.ld + c;
          if (c + 8 <= q.cols) {
            x = *reinterpret_cast<const u32x4_u*>(s);
          } else {
#pragma unroll
            for (int e = 0; e < 8; e++)
              if (c + e < q.cols) x[e >> 1] |= (uint32_t)s[e] << ((e & 1) * 16);
          }
        }
        *reinterpret_cast<u32x4*>(dst + r * q.cols_out + c) = x;
      }
    return;
  }
  const int64_t i = (int64_t)id * 256 + threadIdx.x;
  if (i < j.vn_out) j.vdst[i] = i < j.vn ? j.vsrc[i] : 0.0f;
}

template <bool P_RM, bool Q_RM, int EPI, int BK, int NS, bool RAG = false, bool CRAG = false>
void launch(FastParams p, hipStream_t s) {
  static OnceFlags configured;   // the dynamic LDS limit is raised once per kernel and device
  auto kern = gemm_bf16_kernel<P_RM, Q_RM, EPI, BK, NS, RAG, CRAG>;
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kLdsBytes, &configured)) return;
  DeviceInfo di;
  if (!device_info(&di)) return;
  // persistent: at most one workgroup per CU (the LDS footprint allows no more); a multiple of the die count
  // whenever the tile count is, so that every die gets the same number
  if (p.ldc == 0) p.ldc = p.I;
  if (p.pstride == 0) p.pstride = (int64_t)p.I * p.J;
  const int ntiles = p.tiles_i * p.tiles_j;
  int wgs = di.cus / p.split;
  if (wgs < di.xcds) wgs = di.xcds;
  if (wgs > ntiles) wgs = ntiles;
  p.xcds = 1;
  if (di.xcds > 1 && ntiles % di.xcds == 0 && wgs >= di.xcds) {
    wgs -= wgs % di.xcds;
    p.xcds = di.xcds;
  }
  const dim3 grid((unsigned)wgs, (unsigned)p.split);
  hipLaunchKernelGGL(kern, grid, dim3(256), kLdsBytes, s, p);
}

// Pipeline shape per contraction (slice width, stages): 64 x 2 or 32 x 4, both 128 KB of LDS.
#ifndef FDL_F1_BK
#define FDL_F1_BK 64
#endif
#ifndef FDL_B3_BK
#define FDL_B3_BK 32
#endif
#ifndef FDL_B4_BK
#define FDL_B4_BK 32
#endif
constexpr int kF1BK = FDL_F1_BK, kB3BK = FDL_B3_BK, kB4BK = FDL_B4_BK;
constexpr int stages_of(int bk) { return kLdsStages / (2 * kTile * bk * 2); }

// ragged_j: J may be any number from kMinRaggedRows up (F1, B3: J = M); otherwise a multiple of the tile
constexpr int64_t kMinRaggedRows = 128;
bool dims_ok(int64_t I, int64_t J, int64_t R, int bk, bool ragged_j = false) {
  const int64_t tj = (J + kTile - 1) / kTile;
  return I > 0 && J > 0 && R > 0 && I % kTile == 0 && (ragged_j ? J >= kMinRaggedRows : J % kTile == 0) &&
         R % (stages_of(bk) * bk) == 0 && I <= (1 << 24) && J <= (1 << 24) && (I / kTile) * tj <= (1 << 30);
}

}  // namespace

bool fast_f1_supported(int64_t M, int64_t K, int64_t N) { return dims_ok(N, M, K, kF1BK, true); }
bool fast_b3_supported(int64_t M, int64_t K, int64_t N) { return dims_ok(K, M, N, kB3BK, true); }
// dW on the fast kernel: the whole reduction if M is a whole number of pipeline rounds, else its first
// fast_b4_rows(M) rows (the caller adds the remaining rows' contribution)
int64_t fast_b4_rows(int64_t M) { const int64_t u = (int64_t)kB4BK * stages_of(kB4BK); return M / u * u; }
bool fast_b4_supported(int64_t M, int64_t K, int64_t N) {
  return fast_b4_rows(M) >= 128 && dims_ok(K, N, fast_b4_rows(M), kB4BK);
}
size_t fast_f1_tail_bytes(int64_t M, int64_t K) { return M % kTile ? (size_t)kTile * K * 2 : 0; }

// ---- padded mode: N and K not both multiples of the tile ---------------------------------------------------------
// The contractions then run on the same kernels with N and K rounded up to the tile: the weights are copied into a
// zero-padded [Np][Kp] matrix (small: it is the only operand that is always copied whole), the bias into a padded vector,
// dZ is laid out with pitch Np and zero surplus columns, and the kernels leave the surplus output columns and rows
// unstored.  X enters in one of two ways:
//   through a copy with pitch Kp, zeros around it and whole row tiles (M K elements read and written once, against three
//     contractions at six to eight times the generic kernel's rate); the rows behind dZ's last are cleared up to a pipeline
//     round, so that dW needs no remainder.  Everywhere but where
//   K is a multiple of the forward pass's pipeline round (128), or the static entry point has no room for the copy and K is
//     a multiple of 8 and at least 128: as it is.  Its last row tile comes from a copy with one spare row, because rows may
//     be read past their end (the surplus meets the weights' zeros: an infinity there makes the row before it NaN, which is
//     why the copy is preferred), and the dW product leaves the last rows to the generic kernel.
int64_t fast_pad_dim(int64_t n) { return (n + kTile - 1) / kTile * kTile; }
bool fast_padded_supported(int64_t M, int64_t K, int64_t N) {
  if (M < kMinRaggedRows || N < 8) return false;
  if (N % kTile == 0 && K % kTile == 0) return false;     // nothing to pad: the plain fast path applies
  const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K), tj = (M + kTile - 1) / kTile;
  if (Np > (1 << 24) || Kp > (1 << 24) || M > (1 << 24) || (Np / kTile) * tj > (1 << 30) || (Kp / kTile) * tj > (1 << 30) ||
      (Np / kTile) * (Kp / kTile) > (1 << 30))
    return false;
  if (N % 8 == 0 && K % 8 == 0 && K >= 128) return true;
  // odd rows: not where the padding is most of the work, nor where the copies' launches are
  return Np * Kp <= 6 * N * K && M * N * K >= kStageFromWork;
}
bool fast_padded_stages_x(int64_t K) { return K % (stages_of(kF1BK) * kF1BK) != 0; }
// X as it is although rows are read past their end: K >= 128, so that such a read ends inside the next row (Kp <= 2 K)
bool fast_padded_can_skip_copy(int64_t K) { return K % 8 == 0 && K >= 128; }
size_t fast_padded_tail_bytes(int64_t K) { return (size_t)(kTile + 1) * K * 2; }
// Rows of X's copy and of dZ, and of dW's reduction over them: whole row tiles, and from 4096 rows a multiple of 512 - the
// reduction is split into equal parts of whole pipeline rounds, and 10000 rows make 79 of those, a prime number (Linear+ReLU
// 10000 x 1000 x 3000: 380 us, 334 with 80 rounds).
int64_t fast_padded_rows(int64_t M) { const int64_t u = M >= 4096 ? 512 : kTile; return (M + u - 1) / u * u; }
// rows of the dW reduction the fast kernel covers in padded mode (X as it is: where it is read past the end of its rows
// the last row it touches must have a successor)
int64_t fast_padded_b4_rows(int64_t M, int64_t K) {
  const int64_t u = (int64_t)kB4BK * stages_of(kB4BK);
  if (fast_padded_stages_x(K)) return M >= 4096 ? fast_padded_rows(M) : (M + u - 1) / u * u;
  return (K % kTile ? M - 1 : M) / u * u;
}

void stage_matrix(StageJobs* j, const void* src, int64_t rows, int64_t cols, int64_t ld, void* dst, int64_t rows_out, int64_t cols_out) {
  if (rows_out <= 0) return;
  StageJob& q = j->job[j->count++];
  q.src = src; q.dst = dst; q.rows = rows; q.cols = cols; q.ld = ld; q.rows_out = rows_out; q.cols_out = cols_out;
  const int64_t wanted = (rows_out * (cols_out / 8) + 255) / 256;        // a vector per thread, up to 2048 workgroups
  q.blocks = (int)(wanted < 1 ? 1 : (wanted > 2048 ? 2048 : wanted));
}
void stage_vector(StageJobs* j, const float* src, int64_t n, float* dst, int64_t n_out) {
  j->vsrc = src; j->vdst = dst; j->vn = n; j->vn_out = n_out;
}
void launch_stage(const StageJobs& j, hipStream_t s) {
  int64_t blocks = (j.vn_out + 255) / 256;
  for (int k = 0; k < j.count; k++) blocks += j.job[k].blocks;
  if (blocks > 0) hipLaunchKernelGGL(stage_kernel, dim3((unsigned)blocks), dim3(256), 0, s, j);
}
// the last row tile of X with one spare row, from rows that are read past their end
static void stage_x_tail(StageJobs* j, const void* X, int64_t M, int64_t K, void* xtail, int64_t spare) {
  const int64_t row0 = (M + kTile - 1) / kTile * kTile - kTile;
  stage_matrix(j, static_cast<const bf16_t*>(X) + row0 * K, M - row0, K, K, xtail, kTile + spare, K);
}
// W [N][K] -> Wp [Np][Kp], bias (may be null) -> biasp [Np], and X -> xw: all of it (staged) or its last row tile
void stage_padded(StageJobs* j, int64_t M, int64_t K, int64_t N, bool staged, const void* X, const void* W, const float* bias,
                  void* xw, void* Wp, float* biasp) {
  const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K);
  if (X != nullptr) {
    if (staged) stage_matrix(j, X, M, K, K, xw, fast_padded_rows(M), Kp);
    else stage_x_tail(j, X, M, K, xw, 1);
  }
  stage_matrix(j, W, N, K, K, Wp, Np, Kp);
  if (biasp != nullptr) stage_vector(j, bias, N, biasp, Np);
}

// Wb = W [N][K] in blocks of 32 x 32 (N, K multiples of 64).
void launch_fast_block(int64_t N, int64_t K, const void* W, void* Wb, hipStream_t s) {
  hipLaunchKernelGGL(block32_kernel, dim3((unsigned)(K / 64), (unsigned)(N / 32)), dim3(256), 0, s, (const bf16_t*)W, K, (bf16_t*)Wb);
}

static void launch_xwt_split(FastParams p, bool rag, bool crag, int kind, int split, void* part, int64_t M, int64_t N,
                             const float* bias, const void* aux, void* out, int64_t ldo, hipStream_t s);

// Padded mode: the operands of stage_padded.  kind as launch_fast_xwt; kind 2 writes out [..][Np], the others [M][N].
// split, part: see fast_xwt_split.
void launch_fast_xwt_padded(int kind, int64_t M, int64_t K, int64_t N, bool staged, const void* X, const void* xw, const void* Wp,
                            const float* biasp, const void* aux, void* out, int split, void* part, hipStream_t s) {
  const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K);
  FastParams p = {};
  p.P = (const bf16_t*)Wp; p.ldp = Kp;
  p.Q = (const bf16_t*)(staged ? xw : X); p.ldq = staged ? Kp : K;
  // X as it is: the last row tile always comes from the copy (its rows are read past their end)
  p.Qtail = staged ? nullptr : (const bf16_t*)xw;
  p.C = (bf16_t*)out; p.bias = biasp; p.aux = (const bf16_t*)aux; p.ldc = kind == 2 ? Np : N;
  p.I = (int)N; p.J = (int)M; p.tiles_i = (int)(Np / kTile); p.tiles_j = (int)((M + kTile - 1) / kTile);
  constexpr int NS = stages_of(kF1BK), round = NS * kF1BK;
  p.nkt = (int)((K + round - 1) / round * NS); p.split = 1;
  if (split > 1) { launch_xwt_split(p, true, true, kind, split, part, M, N, biasp, aux, out, p.ldc, s); return; }
  if (kind == 1) launch<false, false, EPI_RELU, kF1BK, NS, true, true>(p, s);
  else if (kind == 2) launch<false, false, EPI_MASK, kF1BK, NS, true, true>(p, s);
  else if (biasp != nullptr) launch<false, false, EPI_BIAS, kF1BK, NS, true, true>(p, s);
  else launch<false, false, EPI_STORE, kF1BK, NS, true, true>(p, s);
}

// out[m][n] = f(sum_k X[m][k] W[n][k] + bias[n]): the forward product (fast_f1_supported shapes).
//   kind 0: plain product (bias may be null: then none is added)      kind 1: max(. , 0)
//   kind 2: aux[m][n] where the sum is positive, else 0
// xtail: fast_f1_tail_bytes(M, K) bytes of scratch when M is not a multiple of 256, unless X itself has readable rows
// up to the next multiple of 256 (x_padded).
// out_blocked (kind 2 only; M, N multiples of 32): out is written in 32 x 32 blocks, as the dX and dW kernels read it best.
void launch_fast_xwt(int kind, int64_t M, int64_t K, int64_t N, const void* X, bool x_padded, const void* W,
                     const float* bias, const void* aux, void* out, bool out_blocked, void* xtail,
                     hipStream_t s, int split, void* part) {
  FastParams p = {};
  p.cblocked = (out_blocked && kind == 2) ? 1 : 0;
  p.P = (const bf16_t*)W; p.Q = (const bf16_t*)X; p.ldp = K; p.ldq = K;
  p.C = (bf16_t*)out; p.bias = bias; p.aux = (const bf16_t*)aux;
  p.I = (int)N; p.J = (int)M; p.tiles_i = (int)(N / kTile); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(K / kF1BK); p.split = 1;
  const bool rag = M % kTile != 0;
  if (rag && !x_padded) {
    p.Qtail = (const bf16_t*)xtail;
    StageJobs j = {};
    stage_x_tail(&j, X, M, K, xtail, 0);
    launch_stage(j, s);
  }
  if (split > 1) { launch_xwt_split(p, rag, false, kind, split, part, M, N, bias, aux, out, N, s); return; }
  constexpr int NS = stages_of(kF1BK);
#define FDL_XWT(EPI)                                                              \
  do {                                                                            \
    if (rag) launch<false, false, EPI, kF1BK, NS, true>(p, s);                    \
    else launch<false, false, EPI, kF1BK, NS, false>(p, s);                       \
  } while (0)
  if (kind == 1) FDL_XWT(EPI_RELU);
  else if (kind == 2) FDL_XWT(EPI_MASK);
  else if (bias != nullptr) FDL_XWT(EPI_BIAS);
  else FDL_XWT(EPI_STORE);
#undef FDL_XWT
}

// out = X W^T with both operands in blocks of 32 x 32, X (the library's own buffer) with its rows padded to whole tiles.  Every slice
// of either is long runs, for which slices of 32 in four stages serve better than slices of 64 in two: the feed-forward block's down
// product 16384 x 11008 x 4096 1115 us from rows 22 KB apart, 935 so, 14 of it the weights' copy.  An X that comes as rows gains nothing
// from blocked weights (inference, us, with / without: 16384 x 4096 x 4096 428 / 408, 32768 x 2048 x 8192 956 / 930,
// 16384 x 11008 x 4096 1187 / 1188; at the shortest
// reduction, K = 128, whole calls of 16384 to 100000 rows, without / with, on average: 256 columns 0.92, 2048 0.97, 4096 and more 0.98 - 1.0).
void launch_fast_xwt_blocked(int64_t M, int64_t K, int64_t N, const void* X, const void* Wb, void* out, hipStream_t s) {
  FastParams p = {};
  p.pblocked = p.qblocked = 1;
  p.P = (const bf16_t*)Wb; p.Q = (const bf16_t*)X; p.ldp = K; p.ldq = K;
  p.C = (bf16_t*)out;
  p.I = (int)N; p.J = (int)M; p.tiles_i = (int)(N / kTile); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(K / kB3BK); p.split = 1;
  constexpr int NS = stages_of(kB3BK);
  if (M % kTile != 0) launch<false, false, EPI_STORE, kB3BK, NS, true>(p, s);
  else launch<false, false, EPI_STORE, kB3BK, NS, false>(p, s);
}

// ---- the forward product with a split reduction ------------------------------------------------------------------
// A batch of a few hundred rows has few output tiles (512 x 4096: 32 on 256 compute units), and each takes its whole
// reduction, about 1.1 us per slice of 64 however few there are.  The parts of a split leave fp32 sums, which a second
// kernel adds in order and finishes.
// Prices, us: a tile's start and end 6, a slice 1.1; a part's with its 256 KB of sums 13, the second kernel 5 and its reading
// at 6 TB/s.  Measured, us, whole / split, K x N and rows: 4096 x 4096: 512 77 / 42, 1024 78 / 58, 2048 82 / 87 (not split);
// 4096 x 1024: 2048 77 / 43, 4096 79 / 62; 2048 x 2048: 1024 42 / 32; 4096 x 512: 4096 77 / 42, 8192 78 / 61.
double fast_xwt_cost(int64_t M, int64_t K, int64_t N, int* split_out) {
  const int64_t tiles = fast_pad_dim(N) / kTile * ((M + kTile - 1) / kTile);
  constexpr int NS = stages_of(kF1BK), round = NS * kF1BK;
  const int64_t rounds_k = (K + round - 1) / round;       // pipeline rounds of the reduction
  int best = 1;
  double best_cost = (double)((tiles + kPlanCUs - 1) / kPlanCUs) * ((double)rounds_k * NS * 1.1 + 6.0);
  for (int split = 2; split <= 16 && tiles * split <= kPlanCUs; split++) {
    if (rounds_k % split) continue;
    const double cost = (double)(rounds_k / split) * NS * 1.1 + 18.0 + (double)split * (double)M * (double)N * 4.0 / 6e6;
    if (cost < 0.9 * best_cost) { best = split; best_cost = cost; }
  }
  if (split_out != nullptr) *split_out = best;
  return best_cost;
}
int fast_xwt_split(int64_t M, int64_t K, int64_t N) {
  int split = 1;
  fast_xwt_cost(M, K, N, &split);
  return split;
}
size_t fast_xwt_part_bytes(int64_t M, int64_t N, int split) { return split > 1 ? (size_t)split * partial_stride(M * N) * 4 : 0; }

namespace {
// out[m][n] = f(the parts' sums + bias[n]), kinds as launch_fast_xwt; out has pitch ldo (kind 2: zeros from N to ldo)
template <int KIND>
__global__ __launch_bounds__(256) void xwt_reduce_kernel(const float* __restrict__ part, int split, int64_t stride, int64_t M,
                                                         int64_t N, const float* __restrict__ bias,
                                                         const bf16_t* __restrict__ aux, bf16_t* __restrict__ out, int64_t ldo) {
  typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
  typedef __bf16 bf16x4_u __attribute__((ext_vector_type(4), aligned(2)));
  const int64_t width = KIND == 2 ? ldo : N, vpr = (width + 3) / 4;
  for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < M * vpr; v += (int64_t)gridDim.x * 256) {
    const int64_t m = v / vpr, n = (v - m * vpr) * 4;
    const int left = N - n > 4 ? 4 : (N - n < 0 ? 0 : (int)(N - n));
    float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const float* src = part + m * N + n;
    if (left == 4) {
#pragma unroll 4
      for (int k = 0; k < split; k++) {            // (four loads in flight)
        const f32x4_u t = *reinterpret_cast<const f32x4_u*>(src + (int64_t)k * stride);
#pragma unroll
        for (int e = 0; e < 4; e++) z[e] += t[e];
      }
    } else {
      for (int k = 0; k < split; k++)
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (e < left) z[e] += src[(int64_t)k * stride + e];
    }
    bf16x4_u o;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float x = z[e] + (bias != nullptr && e < left ? bias[n + e] : 0.0f);
      if (KIND == 2) o[e] = e < left && x > 0.0f ? aux[m * N + n + e] : (bf16_t)0.0f;
      else o[e] = (bf16_t)(KIND == 1 ? (x > 0.0f ? x : 0.0f) : x);
    }
    bf16_t* dst = out + m * ldo + n;
    if (n + 4 <= width) {
      *reinterpret_cast<bf16x4_u*>(dst) = o;
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (n + e < width) dst[e] = o[e];
    }
  }
}
}  // namespace

void launch_xwt_reduce(int kind, int split, const void* part, int64_t stride, int64_t M, int64_t N, const float* bias, const void* aux,
                       void* out, int64_t ldo, hipStream_t s) {
  const int64_t vectors = M * ((ldo + 3) / 4);
  const unsigned blocks = (unsigned)((vectors + 255) / 256 < 4096 ? (vectors + 255) / 256 : 4096);
  auto kern = kind == 1 ? xwt_reduce_kernel<1> : (kind == 2 ? xwt_reduce_kernel<2> : xwt_reduce_kernel<0>);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, s, (const float*)part, split, stride, M, N, bias, (const bf16_t*)aux,
                     (bf16_t*)out, ldo);
}

// split > 1: part holds fast_xwt_part_bytes; p: the product's operands, tiles and sizes (a forward product of the functions
// above, before its epilogue is chosen); crag: any N
static void launch_xwt_split(FastParams p, bool rag, bool crag, int kind, int split, void* part, int64_t M, int64_t N,
                             const float* bias, const void* aux, void* out, int64_t ldo, hipStream_t s) {
  p.bias = nullptr; p.aux = nullptr;
  p.Cpart = (float*)part; p.pstride = partial_stride(M * N); p.split = split; p.nkt /= split;
  constexpr int NS = stages_of(kF1BK);
  if (crag) launch<false, false, EPI_PARTIAL, kF1BK, NS, true, true>(p, s);
  else if (rag) launch<false, false, EPI_PARTIAL, kF1BK, NS, true>(p, s);
  else launch<false, false, EPI_PARTIAL, kF1BK, NS>(p, s);
  launch_xwt_reduce(kind, split, part, p.pstride, M, N, bias, aux, out, ldo, s);
}

// Gated pair of products for the feed-forward block: Hout[m][h] = SiLU(sum_d X[m][d] Wg[h][d]) * (sum_d X[m][d] Wu[h][d]).
// Shapes: H a multiple of 128, D of the pipeline round, M >= 128; ragged M as in launch_fast_xwt.
bool fast_gate_supported(int64_t M, int64_t D, int64_t H) {
  const int64_t tj = (M + kTile - 1) / kTile;
  return M >= kMinRaggedRows && H > 0 && H % 128 == 0 && D > 0 && D % (stages_of(kF1BK) * kF1BK) == 0 && H <= (1 << 24) &&
         M <= (1 << 24) && (H / 128) * tj <= (1 << 30);
}
void launch_fast_gate(int64_t M, int64_t D, int64_t H, const void* X, const void* Wg, const void* Wu, void* Hout, bool out_blocked,
                      void* xtail, hipStream_t s) {
  FastParams p = {};
  p.cblocked = out_blocked ? 1 : 0;    // H a multiple of 32; rows past M are not stored
  p.P = (const bf16_t*)Wg; p.P2 = (const bf16_t*)Wu; p.Q = (const bf16_t*)X; p.ldp = D; p.ldq = D;
  p.C = (bf16_t*)Hout;
  p.I = (int)H; p.J = (int)M; p.tiles_i = (int)(H / 128); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(D / kF1BK); p.split = 1;
  const bool rag = M % kTile != 0;
  if (rag) {
    p.Qtail = (const bf16_t*)xtail;
    StageJobs j = {};
    stage_x_tail(&j, X, M, D, xtail, 0);
    launch_stage(j, s);
  }
  constexpr int NS = stages_of(kF1BK);
  if (rag) launch<false, false, EPI_GATE, kF1BK, NS, true>(p, s);
  else launch<false, false, EPI_GATE, kF1BK, NS, false>(p, s);
}

// Padded: Wgp, Wup [Hp][Dp] zero-padded copies (Hp a multiple of 128, Dp of the pipeline round); X as it is (xw: the copy of
// its last row tile) or as a copy xw with pitch Dp (fast_padded_stages_x); Hout [..][Hp] with zero surplus columns.
int64_t fast_gate_pad_h(int64_t H) { return (H + 127) / 128 * 128; }
int64_t fast_gate_pad_d(int64_t D) { const int64_t u = (int64_t)stages_of(kF1BK) * kF1BK; return (D + u - 1) / u * u; }
void launch_fast_gate_padded(int64_t M, int64_t D, int64_t H, const void* X, const void* xw, const void* Wgp, const void* Wup,
                             void* Hout, hipStream_t s) {
  const int64_t Hp = fast_gate_pad_h(H), Dp = fast_gate_pad_d(D);
  const bool staged = fast_padded_stages_x(D);
  FastParams p = {};
  p.P = (const bf16_t*)Wgp; p.P2 = (const bf16_t*)Wup; p.ldp = Dp;
  p.Q = (const bf16_t*)(staged ? xw : X); p.ldq = staged ? Dp : D;
  p.Qtail = staged ? nullptr : (const bf16_t*)xw;
  p.C = (bf16_t*)Hout; p.ldc = Hp;
  p.I = (int)H; p.J = (int)M; p.tiles_i = (int)(Hp / 128); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(Dp / kF1BK); p.split = 1;
  launch<false, false, EPI_GATE, kF1BK, stages_of(kF1BK), true, true>(p, s);
}
// out [M][D] = G [..][Hp] Wdp^T with Wdp [D rounded up to the tile][Hp]; G has readable rows up to the next row tile
void launch_fast_down_padded(int64_t M, int64_t D, int64_t Hp, const void* G, const void* Wdp, void* out, int split, void* part,
                             hipStream_t s) {
  FastParams p = {};
  p.P = (const bf16_t*)Wdp; p.Q = (const bf16_t*)G; p.ldp = Hp; p.ldq = Hp;
  p.C = (bf16_t*)out;
  p.I = (int)D; p.J = (int)M; p.tiles_i = (int)(fast_pad_dim(D) / kTile); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(Hp / kF1BK); p.split = 1;
  if (split > 1) { launch_xwt_split(p, true, true, 0, split, part, M, D, nullptr, nullptr, out, D, s); return; }
  launch<false, false, EPI_STORE, kF1BK, stages_of(kF1BK), true, true>(p, s);
}
void stage_gate_x(StageJobs* j, const void* X, int64_t M, int64_t D, void* xw) {
  if (fast_padded_stages_x(D)) stage_matrix(j, X, M, D, D, xw, fast_padded_rows(M), fast_gate_pad_d(D));
  else stage_x_tail(j, X, M, D, xw, 1);
}

void launch_fast_b3(int64_t M, int64_t K, int64_t N, const void* dZ, bool dz_blocked, const void* W, void* dX,
                    hipStream_t s) {
  FastParams p = {};
  p.qblocked = dz_blocked ? 1 : 0;
  p.P = (const bf16_t*)W; p.Q = (const bf16_t*)dZ; p.ldp = K; p.ldq = N;
  p.C = (bf16_t*)dX;
  p.I = (int)K; p.J = (int)M; p.tiles_i = (int)(K / kTile); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(N / kB3BK); p.split = 1;
  // ragged M: dZ is the library's own buffer and has readable rows up to the end of the last row tile
  if (M % kTile) launch<true, false, EPI_STORE, kB3BK, stages_of(kB3BK), true>(p, s);
  else launch<true, false, EPI_STORE, kB3BK, stages_of(kB3BK)>(p, s);
}

// Padded mode: dZ [.][Np] with zero surplus columns and readable rows up to the next multiple of 256; Wp [Np][Kp]
void launch_fast_b3_padded(int64_t M, int64_t K, int64_t N, const void* dZ, const void* Wp, void* dX, hipStream_t s) {
  const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K);
  FastParams p = {};
  p.P = (const bf16_t*)Wp; p.Q = (const bf16_t*)dZ; p.ldp = Kp; p.ldq = Np;
  p.C = (bf16_t*)dX;
  p.I = (int)K; p.J = (int)M; p.tiles_i = (int)(Kp / kTile); p.tiles_j = (int)((M + kTile - 1) / kTile);
  p.nkt = (int)(Np / kB3BK); p.split = 1;
  launch<true, false, EPI_STORE, kB3BK, stages_of(kB3BK), true, true>(p, s);
}

// Split of the reduction over M.  One workgroup per compute unit walks the (tile, part) units of its part, so the
// kernel takes ceil(tiles * split / CUs) rounds of M / split rows each: a small dW fills the chip only when split,
// and a dW with a few tiles more than a whole number of rounds (9 x 32 = 288 tiles on 256 compute units: two rounds,
// the second nearly empty) loses up to half its time unless the rounds are made shorter.  Against that stands the
// traffic of the fp32 partial sums (written, read again and summed).  Both are priced with round figures for this
// part - 23 ns per reduction row and round, 4 TB/s for the partial sums - and the cheapest split wins; each part keeps
// at least 512 rows and a whole number of pipeline rounds, and the partial sums at most 512 MB.
int fast_b4_split(int64_t M, int64_t K, int64_t N) {
  const int64_t tiles = ((K + kTile - 1) / kTile) * ((N + kTile - 1) / kTile);
  const int64_t unit = (int64_t)kB4BK * stages_of(kB4BK);   // every part is a whole number of slice groups
  int best = 1;
  double best_cost = 0.0;
  for (int split = 1; split <= 16; split *= 2) {
    if (split > 1 && (M % (split * unit) != 0 || M / split < 512)) break;
    const double partial_bytes = split > 1 ? (double)split * (double)tiles * kTile * kTile * 4.0 : 0.0;
    if (partial_bytes > 512.0 * 1024 * 1024) break;
    const int64_t rounds = (tiles * split + kPlanCUs - 1) / kPlanCUs;
    const double cost = (double)rounds * (double)(M / split) * 23e-9 + 2.0 * partial_bytes / 4e12;
    if (split == 1 || cost < 0.97 * best_cost) { best = split; best_cost = cost; }
  }
  return best;   // M: the rows the fast kernel covers
}

// dW from the first M rows (a whole number of pipeline rounds, see fast_b4_rows).  With split > 1 or extra > 0 the
// kernel writes fp32 partial sums dwpart[0 .. split); the caller may add `extra` more partials behind them (the
// rows the fast kernel does not cover) and then sums them (the backward pass's finishing launch); otherwise dW is final on return.
void launch_fast_b4(int64_t M, int64_t K, int64_t N, int split, int extra, const void* dZ, bool dz_blocked, const void* X,
                    void* dW, void* dwpart, hipStream_t s) {
  FastParams p = {};
  p.qblocked = dz_blocked ? 1 : 0;
  p.P = (const bf16_t*)X; p.Q = (const bf16_t*)dZ; p.ldp = K; p.ldq = N;
  p.C = (bf16_t*)dW; p.Cpart = (float*)dwpart;
  p.I = (int)K; p.J = (int)N; p.tiles_i = (int)(K / kTile); p.tiles_j = (int)(N / kTile);
  p.nkt = (int)(M / kB4BK / split); p.split = split;
  if (split > 1 || extra > 0) launch<true, true, EPI_PARTIAL, kB4BK, stages_of(kB4BK)>(p, s);
  else launch<true, true, EPI_STORE, kB4BK, stages_of(kB4BK)>(p, s);
}

// Padded mode: dZ has pitch Np (zero surplus columns), X pitch ldx (K or, as a copy, Kp); M at most fast_padded_b4_rows.
// With split > 1 or extra > 0 fp32 partial sums as launch_fast_b4, otherwise dW [N][K] is final on return.
void launch_fast_b4_padded(int64_t M, int64_t K, int64_t N, int split, int extra, const void* dZ, const void* X, int64_t ldx,
                           void* dW, void* dwpart, hipStream_t s) {
  const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K);
  FastParams p = {};
  p.P = (const bf16_t*)X; p.Q = (const bf16_t*)dZ; p.ldp = ldx; p.ldq = Np;
  p.C = (bf16_t*)dW; p.Cpart = (float*)dwpart; p.pstride = partial_stride(N * K);
  p.I = (int)K; p.J = (int)N; p.tiles_i = (int)(Kp / kTile); p.tiles_j = (int)(Np / kTile);
  p.nkt = (int)(M / kB4BK / split); p.split = split;
  if (split > 1 || extra > 0) launch<true, true, EPI_PARTIAL, kB4BK, stages_of(kB4BK), true, true>(p, s);
  else launch<true, true, EPI_STORE, kB4BK, stages_of(kB4BK), true, true>(p, s);
}

// dX and dW in one launch (see gemm_bf16_pair_kernel): for shapes where the two outputs together have at most one tile per
// compute unit of the plan's part (kPlanCUs: the split is part of the workspace plan and must not depend on the device).
// The reductions - over N (padded: Np) for dX, over `rows` rows for dW - are split into sa and sb parts, whole pipeline
// rounds of at least 512, so that the workgroups fill the chip and the longer of the two kinds of workgroup is as short as
// possible.  M, N, K: any with padded operands, else K and N multiples of the tile.  Returns false if it does not qualify.
bool fast_pair_plan(int64_t M, int64_t K, int64_t N, int64_t rows, int* sa_out, int* sb_out) {
  static_assert(kB3BK == kB4BK, "one pipeline shape for both");
  const int64_t Np = fast_pad_dim(N), Kp = fast_pad_dim(K), tj = (M + kTile - 1) / kTile;
  const int64_t ta = (Kp / kTile) * tj, tb = (Kp / kTile) * (Np / kTile);
  if (ta + tb > kPlanCUs) return false;
  const int64_t unit = (int64_t)kB3BK * stages_of(kB3BK);
  int best_sa = 0, best_sb = 0;
  int64_t best_len = 0, best_wgs = 0;
  for (int sa = 1; sa <= 16; sa++) {
    if (Np % (sa * unit) || (sa > 1 && Np / sa < 512)) continue;
    for (int sb = 1; sb <= 16; sb++) {
      if (rows % (sb * unit) || (sb > 1 && rows / sb < 512)) continue;
      const int64_t wgs = ta * sa + tb * sb;
      if (wgs > kPlanCUs) break;
      const int64_t len = Np / sa > rows / sb ? Np / sa : rows / sb;     // reduction length of the longest workgroup
      if (best_sa == 0 || len < best_len || (len == best_len && wgs < best_wgs)) {
        best_sa = sa; best_sb = sb; best_len = len; best_wgs = wgs;
      }
    }
  }
  if (best_sa == 0) return false;
  *sa_out = best_sa; *sb_out = best_sb;
  return true;
}

// dxpart: sa fp32 partial sums [M][K] (sa > 1), dwpart: sb [N][K] (sb > 1, or more of the caller's behind them: extra > 0),
// partial_stride elements apart; an unsplit product goes to dX / dW directly.  Wp: W, or its padded copy (ldw); X with
// pitch ldx; dZ with pitch ldz.
void launch_fast_pair(const PairArgs& a, hipStream_t s) {
  const int64_t Np = fast_pad_dim(a.N), Kp = fast_pad_dim(a.K);
  FastParams pa = {}, pb = {};
  pa.qblocked = pb.qblocked = a.dz_blocked ? 1 : 0;
  pa.P = (const bf16_t*)a.W; pa.Q = (const bf16_t*)a.dZ; pa.ldp = a.ldw; pa.ldq = a.ldz; pa.C = (bf16_t*)a.dX; pa.Cpart = (float*)a.dxpart;
  pa.I = (int)a.K; pa.J = (int)a.M; pa.ldc = a.K; pa.pstride = partial_stride(a.M * a.K);
  pa.tiles_i = (int)(Kp / kTile); pa.tiles_j = (int)((a.M + kTile - 1) / kTile);
  pa.nkt = (int)(Np / kB3BK / a.sa); pa.split = a.sa;
  pb.P = (const bf16_t*)a.X; pb.Q = (const bf16_t*)a.dZ; pb.ldp = a.ldx; pb.ldq = a.ldz; pb.C = (bf16_t*)a.dW; pb.Cpart = (float*)a.dwpart;
  pb.I = (int)a.K; pb.J = (int)a.N; pb.ldc = a.K; pb.pstride = partial_stride(a.N * a.K);
  pb.tiles_i = (int)(Kp / kTile); pb.tiles_j = (int)(Np / kTile);
  pb.nkt = (int)(a.rows / kB4BK / a.sb); pb.split = a.sb;
  DeviceInfo di;
  if (!device_info(&di)) return;
  const int na = pa.tiles_i * pa.tiles_j, nb = pb.tiles_i * pb.tiles_j;     // one tile per workgroup
  const bool die_aware = di.xcds > 1 && na % di.xcds == 0 && nb % di.xcds == 0;
  pa.xcds = die_aware ? di.xcds : 1; pb.xcds = pa.xcds;
  const dim3 grid((unsigned)(na * a.sa + nb * a.sb));
  constexpr int NS = stages_of(kB3BK);
  const bool rag = a.M % kTile || a.N % kTile || a.K % kTile, parta = a.sa > 1, partb = a.sb > 1 || a.extra > 0;
#define FDL_PAIR(EA, EB, RAG)                                                                              \
  do {                                                                                                     \
    static OnceFlags configured;                                                                           \
    auto kern = gemm_bf16_pair_kernel<kB3BK, NS, EA, EB, RAG>;                                             \
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kLdsBytes, &configured)) return;          \
    hipLaunchKernelGGL(kern, grid, dim3(256), kLdsBytes, s, pa, pb, na, nb);                               \
  } while (0)
#define FDL_PAIR_RAG(RAG)                                                  \
  do {                                                                     \
    if (parta && partb) FDL_PAIR(EPI_PARTIAL, EPI_PARTIAL, RAG);           \
    else if (parta) FDL_PAIR(EPI_PARTIAL, EPI_STORE, RAG);                 \
    else if (partb) FDL_PAIR(EPI_STORE, EPI_PARTIAL, RAG);                 \
    else FDL_PAIR(EPI_STORE, EPI_STORE, RAG);                              \
  } while (0)
  if (rag) FDL_PAIR_RAG(true);
  else FDL_PAIR_RAG(false);
#undef FDL_PAIR_RAG
#undef FDL_PAIR
}

}  // namespace fdl
