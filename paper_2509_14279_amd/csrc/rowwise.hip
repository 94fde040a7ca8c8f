// Streaming (HBM-bound) phases of the fused dense-layer block: row statistics and normalisation (forward), the LayerNorm/GELU
// gradient row pass with its column partial sums (backward), and the column reduction that finishes dbeta, dgamma, db.
//
// Row reductions follow the idiom of the paper's row-normalisation kernels (appendix "Highlighted CUDA
// Kernels", LayerNorm forward and Llama RMSNorm forward: vector loads, wavefront shuffles, a small LDS
// exchange between wavefronts) with 64-wide wavefronts; the bias-style column sums are laid out so that
// consecutive lanes read consecutive columns (the paper's linear backward bias kernel walks a column with
// stride N instead).
//
// Arithmetic type C is one level above the storage type T: fp64 for fp32 storage, fp32 for bf16 storage.
#include "common.hip.h"
#include "internal.h"

namespace fdl {
namespace {

__device__ __forceinline__ float read_lane(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// ------------------------------------------------------------------------------------------------
// F2 with its own statistics, narrow rows (bf16 storage, N <= 512 CH): a wavefront owns a row and keeps it in
// registers over three sweeps (GELU and sum; deviations and their squares; scale, shift, store), so Zsave is read
// once, no partial statistics pass through memory and, where a wavefront has its row to itself, no barrier separates the
// sweeps.  Lane l holds the 8-element
// vectors c*64 + l, c < CH, of its row (every load and store of a wavefront covers 1 KB of one row); the next
// row's vectors are fetched while the current row is processed.  gamma and beta sit in LDS, permuted so that a
// lane's four 16-byte reads per vector are lane-contiguous.  Workgroups of NT/64 wavefronts walk the rows with
// stride.  WPR > 1: neighbouring wavefronts share a row and exchange their sums through LDS (as a workgroup of 1024
// threads per row the same normalisation of 4096 x 16384 took 66 - 89 us: its two reductions stop every wavefront of the
// compute unit).  WPR = 8, rows above 16384: gamma and beta do not fit in LDS and are read from the caches at each row
// (LayerNorm of 4096 x 32768: 105 us, 176 with the row reread from the caches for each sweep; x 30003: 163, 293).
// FIT_FULL: N == 512 CH WPR, every lane holds every vector, and loads and stores go past the caches (non-temporal).
// FIT_VECTORS (N % 8 == 0): the vectors past the end of the row
// are fetched from a clamped address, masked to zero (GELU(0) = 0 adds nothing to the sum), left out of the squared
// deviations and never stored; the code stays free of divergent branches either way.  FIT_ANY: rows start at any element
// and end inside a vector - the same 16-byte loads and stores from element-aligned addresses (the hardware splits what
// straddles a line), the row's last, partial vector element by element by the one lane that holds it.
// ACT selects what is normalised: ACT_GELU the GELU of the input (the block's second forward phase; Z and Y may then
// be the same buffer - a lane reads its part of a row before it writes it - so they are not declared restrict),
// ACT_NONE the input itself (stand-alone LayerNorm forward), ACT_RMS the input without mean subtraction and without
// beta (RMSNorm forward: y = x (mean(x^2) + eps)^-1/2 w; mean and rstd are not written).
enum { ACT_GELU = 0, ACT_NONE = 1, ACT_RMS = 2 };
enum { FIT_FULL = 0, FIT_VECTORS = 1, FIT_ANY = 2 };
// gamma and beta of 512 vectors' columns take 4 KB per 64 vectors
constexpr bool affine_in_lds(int groups) { return groups <= 32; }
template <int CH, int FIT, int NT, int ACT, int WPR>
__global__ __launch_bounds__(NT) void f2_rows_kernel(int64_t M, int64_t N, float eps, const bf16_t* Z,
                                                      const float* __restrict__ gamma, const float* __restrict__ beta,
                                                      bf16_t* Y, float* __restrict__ mean,
                                                      float* __restrict__ rstd, int stretches) {
  // products are formed once and reused (fusing GELU's final multiplication into each later use would keep
  // both of its factors alive for every element of the row); the fused operations wanted are written out
#pragma clang fp contract(off)
  constexpr bool FULL = FIT == FIT_FULL, ANY = FIT == FIT_ANY;
  constexpr bool kStretches = FULL && WPR > 1;
  // The block's statistics (ACT_GELU; saved, and multiplied into everything the backward pass forms): fp32 inside a vector -
  // up to 1024 columns, where a row has little other work, inside a row of 16 lanes - and fp64 from there on, as is rstd.
  // (fp32 throughout, inference 65536 x 128 x 512: 61.1 us, so 61.9, fp64 from the vector on 64.2; 4096 x 128 x 16384: 108.8,
  // now 110.9; no difference at 4096 and 8192 columns.)  The stand-alone norms keep fp32 (LayerNorm 65536 x 512 22.5 us, 24.3).
  constexpr bool kWide = ACT == ACT_GELU, kShort = CH * WPR <= 2;
  typedef typename std::conditional<kWide && !kShort, double, float>::type sum_t;     // of a lane
  typedef typename std::conditional<kWide, double, float>::type stat_t;               // of a row
  typedef __bf16 bf16x8_u __attribute__((ext_vector_type(8), aligned(2)));
  typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(2)));
  extern __shared__ f32x4 gb[];   // [CH * WPR][4][64]: gamma[0:4], gamma[4:8], beta[0:4], beta[4:8] of each vector
  __shared__ stat_t pair[2][NT / 64];
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  typedef GaussTable<false> GT;
  typedef __attribute__((address_space(3))) float lds_float;
  constexpr bool kAffineLds = affine_in_lds(CH * WPR);
  float* htab = reinterpret_cast<float*>(gb + (kAffineLds ? CH * WPR * 4 * 64 : 0));     // Phi - 1/2 for every bf16 magnitude
  const uint32_t horg = GT::origin((uint32_t)(uintptr_t)(const lds_float*)htab);
  if (ACT == ACT_GELU) GT::build(htab, threadIdx.x, NT);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: row addresses stay scalar
  const int nvec = (int)(N >> 3);              // whole vectors of a row
  const int rest = ANY ? (int)(N & 7) : 0;     // elements of its partial one
  for (int idx = threadIdx.x; idx < (kAffineLds ? CH * WPR * 64 : 0); idx += NT) {
    const int c = idx >> 6, l = idx & 63;
    if (ANY && idx >= nvec) {
      const int have = idx == nvec ? rest : 0;
      float* dst = reinterpret_cast<float*>(gb);
      for (int e = 0; e < 8; e++) {
        dst[((c * 4 + (e >> 2)) * 64 + l) * 4 + (e & 3)] = e < have ? gamma[(int64_t)idx * 8 + e] : 0.0f;
        if (ACT != ACT_RMS) dst[((c * 4 + 2 + (e >> 2)) * 64 + l) * 4 + (e & 3)] = e < have ? beta[(int64_t)idx * 8 + e] : 0.0f;
      }
      continue;
    }
    const int64_t src = (int64_t)(idx < nvec ? idx : nvec - 1) * 8;
    gb[(c * 4 + 0) * 64 + l] = *reinterpret_cast<const f32x4*>(gamma + src);
    gb[(c * 4 + 1) * 64 + l] = *reinterpret_cast<const f32x4*>(gamma + src + 4);
    if (ACT != ACT_RMS) {
      gb[(c * 4 + 2) * 64 + l] = *reinterpret_cast<const f32x4*>(beta + src);
      gb[(c * 4 + 3) * 64 + l] = *reinterpret_cast<const f32x4*>(beta + src + 4);
    }
  }
  __syncthreads();
  // A workgroup's rows: every gridDim.x-th group of kRows, or (stretches > 1, of which the grid is a multiple) the same within its own
  // stretch of them.
  constexpr int kRows = NT / 64 / WPR;
  int64_t first = (int64_t)blockIdx.x * kRows, nw = (int64_t)gridDim.x * kRows, end = M;
  if (kStretches && stretches > 1) {
    const int64_t len = (M + (int64_t)stretches * kRows - 1) / ((int64_t)stretches * kRows) * kRows;
    const int64_t at = (int64_t)(blockIdx.x % (unsigned)stretches) * len;
    first = at + (int64_t)(blockIdx.x / (unsigned)stretches) * kRows;
    nw = (int64_t)(gridDim.x / (unsigned)stretches) * kRows;
    end = at + len < M ? at + len : M;
  }
  const stat_t inv_n = (stat_t)1 / (stat_t)N;
  const int sub = WPR == 1 ? 0 : wave % WPR;   // which part of every vector group this wavefront of the row holds
  // sum k of this trip's row over the wavefronts that share it (row_sum_slot: why one barrier each is enough)
  int trip = 0;
  auto row_sum = [&](sum_t part, int k) -> stat_t {
    stat_t x;
    if constexpr (kWide && kShort) {
      part = row16_sum(part);
      x = ((double)read_lane(part, 0) + (double)read_lane(part, 16)) + ((double)read_lane(part, 32) + (double)read_lane(part, 48));
    } else {
      x = wave_sum(part);
    }
    if constexpr (WPR > 1) {
      const int slot = row_sum_slot(ACT == ACT_RMS ? 1 : 2, trip, k);
      if (lane == 0) pair[slot][wave] = x;
      __syncthreads();
      x = pair[slot][wave - sub];
#pragma unroll
      for (int w = 1; w < WPR; w++) x += pair[slot][wave - sub + w];
    }
    return x;
  };
  // per-lane element offset of vector c inside a row, and whether the row has that vector (FIT_ANY: how many of its
  // elements)
  int voff[CH], have[CH];
  uint32_t keep[CH];
#pragma unroll
  for (int c = 0; c < CH; c++) {
    const int vi = (c * WPR + sub) * 64 + lane;
    voff[c] = (FULL || vi < nvec ? vi : (ANY ? 0 : nvec - 1)) * 8;
    keep[c] = (FULL || vi < nvec) ? 0xffffffffu : 0u;
    have[c] = vi < nvec ? 8 : (vi == nvec ? rest : 0);
  }

  u32x4 raw[CH];
  // vector c of row r (past the last row: a harmless re-read of the last one, never used)
  auto fetch1 = [&](int c, const bf16_t* zr) {
    if (FULL) {
      // scalar base per vector + one shared per-lane offset (the immediate offset field reaches only 4 KB)
      const bf16_t* zc = zr + (c * WPR + sub) * 512;
      asm("" : "+s"(zc));
      raw[c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(zc + lane * 8));
    } else if (ANY) {
      if (have[c] == 8) {
        raw[c] = *reinterpret_cast<const u32x4_u*>(zr + voff[c]);
      } else {
        raw[c] = u32x4{0u, 0u, 0u, 0u};
        if (have[c] != 0) {
          bf16x8 t;
#pragma unroll
          for (int v = 0; v < 8; v++) t[v] = v < have[c] ? zr[nvec * 8 + v] : (bf16_t)0.0f;
          raw[c] = __builtin_bit_cast(u32x4, t);
        }
      }
    } else {
      raw[c] = *reinterpret_cast<const u32x4*>(zr + voff[c]);
    }
  };
  int64_t row = first + wave / WPR;
  {
    const bf16_t* zr = Z + (row < M ? row : M - 1) * N;
#pragma unroll
    for (int c = 0; c < CH; c++) fetch1(c, zr);
  }
  // Where wavefronts share rows, those of a workgroup stay together (barriers): the last trip may find some of them past
  // the last row, which they then redo without storing.
  for (int64_t lead = first; WPR == 1 ? row < end : lead < end; row += nw, lead += nw, trip++) {
    const bool live = WPR == 1 || row < end;
    float a[CH][8];
    sum_t sum = 0;
    const bf16_t* znext = Z + (row + nw < M ? row + nw : M - 1) * N;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      float sum8 = kWide ? 0.0f : (float)sum;          // (fp32 throughout: one chain over the lane's vectors)
#pragma unroll
      for (int h = 0; h < 4; h++) {
        const uint32_t w = (FULL || ANY) ? raw[c][h] : (raw[c][h] & keep[c]);
        const float z0 = __builtin_bit_cast(float, w << 16);                        // bf16 -> fp32 is a 16-bit shift
        const float z1 = __builtin_bit_cast(float, w & 0xffff0000u);
        if (ACT == ACT_GELU) {
          const float h0 = *(const lds_float*)(uintptr_t)GT::address_of(w, horg);
          const float h1 = *(const lds_float*)(uintptr_t)GT::address_of(w >> 16, horg);
          a[c][2 * h] = z0 * (0.5f + GT::with_sign_of(h0, z0));                     // GELU(z) = z Phi(z)
          a[c][2 * h + 1] = z1 * (0.5f + GT::with_sign_of(h1, z1));
        } else {
          a[c][2 * h] = z0;
          a[c][2 * h + 1] = z1;
        }
        if (ACT == ACT_RMS) {
          sum8 = __builtin_fmaf(z0, z0, sum8);
          sum8 = __builtin_fmaf(z1, z1, sum8);
        } else {
          sum8 += a[c][2 * h];
          sum8 += a[c][2 * h + 1];
        }
      }
      sum = kWide ? sum + (sum_t)sum8 : (sum_t)sum8;
      // One vector at a time (interleaving all of a row's evaluations would keep their temporaries alive), and as
      // soon as a vector is unpacked its registers take the same vector of the wavefront's next row: the loads
      // trickle out through the whole first sweep and have the rest of the row's work to arrive, while a row of
      // packed values and a row of fp32 values are all a lane ever holds.
      __builtin_amdgcn_sched_barrier(0);
      fetch1(c, znext);
      __builtin_amdgcn_sched_barrier(0);
    }
    float rs;
    if (ACT == ACT_RMS) {
      rs = 1.0f / __builtin_sqrtf(row_sum(sum, 0) * inv_n + eps);   // masked vectors hold zeros: they add nothing
    } else {
      const float mu = (float)(row_sum(sum, 0) * inv_n);
      sum_t m2 = 0;
#pragma unroll
      for (int c = 0; c < CH; c++) {
        float sq8 = kWide ? 0.0f : (float)m2;
#pragma unroll
        for (int v = 0; v < 8; v++) {
          const float d = a[c][v] - mu;
          a[c][v] = FULL ? d : ((ANY ? v < have[c] : keep[c] != 0u) ? d : 0.0f);
          sq8 = __builtin_fmaf(a[c][v], a[c][v], sq8);
        }
        m2 = kWide ? m2 + (sum_t)sq8 : (sum_t)sq8;
      }
      const stat_t var = row_sum(m2, 1) * inv_n + (stat_t)eps;
      if constexpr (kWide) rs = inv_sqrt(var);
      else rs = 1.0f / __builtin_sqrtf(var);
      if (lane == 0 && sub == 0 && live) { mean[row] = mu; rstd[row] = rs; }
    }
    if (!live) continue;
    bf16_t* yr = Y + row * N;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int cg = c * WPR + sub;
      f32x4 g0, g1, b0 = {}, b1 = {};
      if constexpr (kAffineLds) {
        g0 = gb[(cg * 4 + 0) * 64 + lane], g1 = gb[(cg * 4 + 1) * 64 + lane];
        if (ACT != ACT_RMS) b0 = gb[(cg * 4 + 2) * 64 + lane], b1 = gb[(cg * 4 + 3) * 64 + lane];
      } else if (!ANY || have[c] == 8) {
        // (voff of a vector past the end is that of one inside)
        const int at = FULL ? (cg * 64 + lane) * 8 : voff[c];
        g0 = *reinterpret_cast<const f32x4*>(gamma + at), g1 = *reinterpret_cast<const f32x4*>(gamma + at + 4);
        if (ACT != ACT_RMS) b0 = *reinterpret_cast<const f32x4*>(beta + at), b1 = *reinterpret_cast<const f32x4*>(beta + at + 4);
      } else {
#pragma unroll
        for (int v = 0; v < 4; v++) {
          g0[v] = v < have[c] ? gamma[nvec * 8 + v] : 0.0f;
          g1[v] = v + 4 < have[c] ? gamma[nvec * 8 + v + 4] : 0.0f;
          if (ACT != ACT_RMS) {
            b0[v] = v < have[c] ? beta[nvec * 8 + v] : 0.0f;
            b1[v] = v + 4 < have[c] ? beta[nvec * 8 + v + 4] : 0.0f;
          }
        }
      }
      bf16x8 o;
      if (ACT == ACT_RMS) {
#pragma unroll
        for (int v = 0; v < 4; v++) {
          o[v] = (bf16_t)(a[c][v] * rs * g0[v]);
          o[v + 4] = (bf16_t)(a[c][v + 4] * rs * g1[v]);
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; v++) {
          o[v] = (bf16_t)__builtin_fmaf(a[c][v] * rs, g0[v], b0[v]);
          o[v + 4] = (bf16_t)__builtin_fmaf(a[c][v + 4] * rs, g1[v], b1[v]);
        }
      }
      if (FULL) {
        bf16_t* yc = yr + (c * WPR + sub) * 512;
        asm("" : "+s"(yc));
        __builtin_nontemporal_store(o, reinterpret_cast<bf16x8*>(yc + lane * 8));
      } else if (keep[c]) {
        if (ANY) *reinterpret_cast<bf16x8_u*>(yr + voff[c]) = o;
        else *reinterpret_cast<bf16x8*>(yr + voff[c]) = o;
      } else if (ANY && have[c] != 0) {
#pragma unroll
        for (int v = 0; v < 8; v++)
          if (v < have[c]) yr[nvec * 8 + v] = o[v];
      }
      __builtin_amdgcn_sched_barrier(0);   // keep the LDS reads of later vectors from being hoisted (registers)
    }
  }
}

// ------------------------------------------------------------------------------------------------
// sum of two values over a workgroup of NW wavefronts; `red` is this call's LDS slot ([NW][2] of C)
template <class C, int NW> __device__ __forceinline__ void wg_sum2(C& a, C& b, C (*red)[2]) {
  a = wave_sum(a);
  b = wave_sum(b);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[wave][0] = a; red[wave][1] = b; }
  __syncthreads();
  if constexpr (sizeof(C) == 4 && NW <= 16) {
    // lane w of every row of 16 lanes takes wavefront w's pair; one row sum finishes both totals
    const int l = threadIdx.x & 15;
    a = l < NW ? red[l < NW ? l : 0][0] : (C)0;
    b = l < NW ? red[l < NW ? l : 0][1] : (C)0;
    a = row16_sum(a);
    b = row16_sum(b);
  } else {
    a = red[0][0];
    b = red[0][1];
#pragma unroll
    for (int w = 1; w < NW; w++) { a += red[w][0]; b += red[w][1]; }
  }
}

// the same over WPR neighbouring wavefronts, from wavefront `w0` of the workgroup on (WPR = 1: no barrier)
template <class C, int WPR> __device__ __forceinline__ void row_sum2(C& a, C& b, C (*red)[2], int w0) {
  a = wave_sum(a);
  b = wave_sum(b);
  if constexpr (WPR > 1) {
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { red[wave][0] = a; red[wave][1] = b; }
    __syncthreads();
    a = red[w0][0];
    b = red[w0][1];
#pragma unroll
    for (int w = 1; w < WPR; w++) { a += red[w0 + w][0]; b += red[w0 + w][1]; }
  }
}

// nv of V consecutive column sums of a thread to memory, 16 bytes at a time from an element-aligned address (one 4-byte
// store per column and wavefront touches sixteen lines for 256 bytes: a workgroup's 3 N sums took longer than a row)
template <class C, int V> __device__ __forceinline__ void store_columns(C* p, const C (&a)[V], int nv) {
  constexpr int W = 16 / (int)sizeof(C) < V ? 16 / (int)sizeof(C) : V;
  typedef C vec_t __attribute__((ext_vector_type(W), aligned(sizeof(C))));
  if (nv == V) {
#pragma unroll
    for (int h = 0; h < V / W; h++) {
      vec_t t;
#pragma unroll
      for (int e = 0; e < W; e++) t[e] = a[h * W + e];
      *reinterpret_cast<vec_t*>(p + h * W) = t;
    }
  } else {
#pragma unroll
    for (int v = 0; v < V; v++)
      if (v < nv) p[v] = a[v];
  }
}

// A row's vectors of 16 bytes.  ANY: rows start at any element and end inside a vector - the same 16-byte accesses from
// element-aligned addresses (the hardware splits what straddles a line), the last, partial vector element by element.
template <class T, bool ANY, int V = 16 / (int)sizeof(T)> struct RawVec;
template <> struct RawVec<float, false> { typedef f32x4 type; };
template <> struct RawVec<bf16_t, false> { typedef bf16x8 type; };
template <> struct RawVec<float, true> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct RawVec<bf16_t, true> { typedef __bf16 type __attribute__((ext_vector_type(8), aligned(2))); };
template <class T> struct RawVec<T, true, 1> { typedef T type __attribute__((ext_vector_type(1))); };
template <> struct RawVec<bf16_t, false, 4> { typedef __bf16 type __attribute__((ext_vector_type(4))); };
template <> struct RawVec<bf16_t, true, 4> { typedef __bf16 type __attribute__((ext_vector_type(4), aligned(2))); };
template <> struct RawVec<float, false, 8> { typedef float type __attribute__((ext_vector_type(8), aligned(16))); };
template <> struct RawVec<float, true, 8> { typedef float type __attribute__((ext_vector_type(8), aligned(4))); };

template <class T, bool ANY, int V = 16 / (int)sizeof(T)>
__device__ __forceinline__ typename RawVec<T, ANY, V>::type raw_load(const T* p, int nv) {
  typedef typename RawVec<T, ANY, V>::type raw_t;
  if (!ANY || nv == V) return __builtin_nontemporal_load(reinterpret_cast<const raw_t*>(p));
  raw_t r;
#pragma unroll
  for (int v = 0; v < V; v++) r[v] = v < nv ? p[v] : (T)0.0f;
  return r;
}
// the same without the streaming hint (the two-kernel path reads its rows twice)
template <class T, bool ANY>
__device__ __forceinline__ typename RawVec<T, ANY>::type row_load(const T* p, int nv) {
  typedef typename RawVec<T, ANY>::type raw_t;
  constexpr int V = 16 / (int)sizeof(T);
  if (!ANY || nv == V) return *reinterpret_cast<const raw_t*>(p);
  raw_t r;
#pragma unroll
  for (int v = 0; v < V; v++) r[v] = v < nv ? p[v] : (T)0.0f;
  return r;
}
template <class T, bool ANY> __device__ __forceinline__ void row_store(T* p, typename RawVec<T, ANY>::type o, int nv) {
  typedef typename RawVec<T, ANY>::type raw_t;
  constexpr int V = 16 / (int)sizeof(T);
  if (!ANY || nv == V) {
    *reinterpret_cast<raw_t*>(p) = o;
  } else {
#pragma unroll
    for (int v = 0; v < V; v++)
      if (v < nv) p[v] = o[v];
  }
}
// nv elements of the row, then zeros up to the end of the pitch (left: elements from here to there): the surplus columns
// of a padded dZ enter the contractions that read it
template <class T, bool ANY, int V = 16 / (int)sizeof(T)>
__device__ __forceinline__ void raw_store(T* p, typename RawVec<T, ANY, V>::type o, int nv, int64_t left) {
  typedef typename RawVec<T, ANY, V>::type raw_t;
  if (!ANY || left >= V) {
    __builtin_nontemporal_store(o, reinterpret_cast<raw_t*>(p));
  } else {
#pragma unroll
    for (int v = 0; v < V; v++)
      if (v < left) p[v] = o[v];
  }
}

// B1a (two-kernel path, rows too long for one workgroup's registers): c1_i = mean_j g_ij, c2_i = mean_j g_ij Ahat_ij with
// g = dY gamma.
template <class T, bool ANY>
__global__ __launch_bounds__(256) void b1a_kernel(int64_t M, int64_t N, const T* __restrict__ dY,
                                                  const T* __restrict__ Z, const float* __restrict__ gamma,
                                                  const float* __restrict__ mean, const float* __restrict__ rstd,
                                                  typename ComputeOf<T>::type* __restrict__ c12) {
  typedef typename ComputeOf<T>::type C;
  constexpr int V = 16 / (int)sizeof(T);
  __shared__ C red[2][4][2];
  ActTable<T, false, 256> tab;
  tab.build();
  int par = 0;
  for (int64_t row = blockIdx.x; row < M; row += gridDim.x, par ^= 1) {
    const C mu = (C)mean[row], rs = (C)rstd[row];
    C s1 = 0, s2 = 0;
    for (int64_t col = (int64_t)threadIdx.x * V; col < N; col += 256 * V) {
      const int nv = !ANY || N - col > V ? V : (int)(N - col);
      const auto dy = row_load<T, ANY>(dY + row * N + col, nv);
      const auto z = row_load<T, ANY>(Z + row * N + col, nv);
      float gm[V];
      if (nv == V) {
#pragma unroll
        for (int v = 0; v < V; v++) gm[v] = gamma[col + v];
      } else {
#pragma unroll
        for (int v = 0; v < V; v++) gm[v] = v < nv ? gamma[col + v] : 0.0f;
      }
      C a[V];
      tab.template gelu<V>(z, a);
#pragma unroll
      for (int v = 0; v < V; v++) {
        const C g = (C)to_f32<T>(dy[v]) * (C)gm[v];
        const C ah = (a[v] - mu) * rs;
        s1 += g;
        s2 += g * ah;
      }
    }
    wg_sum2<C, 4>(s1, s2, red[par]);
    if (threadIdx.x == 0) { c12[row] = s1 / (C)N; c12[M + row] = s2 / (C)N; }
  }
}

// B1b (two-kernel path): dZ and column partials, given c1 and c2.
template <class T, bool ANY>
__global__ __launch_bounds__(256) void b1b_kernel(int64_t M, int64_t N, int64_t ldz, int rows_per_group, int strips,
                                                  const T* __restrict__ dY, const T* __restrict__ Z,
                                                  const float* __restrict__ gamma, const float* __restrict__ mean,
                                                  const float* __restrict__ rstd,
                                                  const typename ComputeOf<T>::type* __restrict__ c12,
                                                  T* __restrict__ dZ, typename ComputeOf<T>::type* __restrict__ colpart) {
  typedef typename ComputeOf<T>::type C;
  typedef typename RawVec<T, ANY>::type raw_t;
  constexpr int V = 16 / (int)sizeof(T);
  const int strip = blockIdx.x % strips;
  const int64_t grp = blockIdx.x / strips;
  const int64_t col = ((int64_t)strip * 256 + threadIdx.x) * V;
  ActTable<T, true, 256> tab;
  tab.build();
  // (threads past the end of the row stay: their lanes hold scalars of the group's rows)
  const int nv = col >= N ? 0 : (!ANY || N - col > V ? V : (int)(N - col));
  C gm[V], accb[V], accg[V], accz[V];
#pragma unroll
  for (int v = 0; v < V; v++) { gm[v] = v < nv ? (C)gamma[col + v] : (C)0; accb[v] = 0; accg[v] = 0; accz[v] = 0; }
  const int64_t r0 = grp * rows_per_group;
  int64_t r1 = r0 + rows_per_group;
  if (r1 > M) r1 = M;
  // lane l holds the four scalars of row r0 + 64 k + l (read row by row they would be scalar loads, which every wait for
  // the table's LDS reads waits for)
  const int lane = threadIdx.x & 63;
  float lmu = 0.0f, lrs = 0.0f;
  C lc1 = 0, lc2 = 0;
  // two rows of loads in flight
  raw_t rdy[2], rz[2];
#pragma unroll
  for (int v = 0; v < V; v++) { rdy[0][v] = rdy[1][v] = (T)0.0f; rz[0][v] = rz[1][v] = (T)0.0f; }
  auto fetch = [&](int k, int64_t r) {
    if (r < r1 && nv > 0) {
      rdy[k] = row_load<T, ANY>(dY + r * N + col, nv);
      rz[k] = row_load<T, ANY>(Z + r * N + col, nv);
    }
  };
  auto process = [&](int k, int64_t r) {
    const int at = (int)(r - r0) & 63;
    if (at == 0) {
      const int64_t q = r + lane < M ? r + lane : M - 1;
      lmu = mean[q]; lrs = rstd[q]; lc1 = c12[q]; lc2 = c12[M + q];
    }
    const C mu = (C)read_lane(lmu, at), rs = (C)read_lane(lrs, at), c1 = read_lane(lc1, at), c2 = read_lane(lc2, at);
    raw_t o;
    C Phi[V], zphi[V];
    tab.template eval<V>(rz[k], Phi, zphi);
#pragma unroll
    for (int v = 0; v < V; v++) {
      const C z = (C)to_f32<T>(rz[k][v]), dy = (C)to_f32<T>(rdy[k][v]);
      const C ah = (z * Phi[v] - mu) * rs;
      C dz = rs * (dy * gm[v] - c1 - ah * c2) * (Phi[v] + zphi[v]);
      if (ANY) dz = v < nv ? dz : (C)0;
      accb[v] += dy;
      accg[v] += dy * ah;
      accz[v] += dz;
      o[v] = to_storage<T, C>(dz);
    }
    fetch(k, r + 2);
    if (nv > 0) row_store<T, ANY>(dZ + r * ldz + col, o, nv);
  };
  fetch(0, r0);
  fetch(1, r0 + 1);
  for (int64_t r = r0; r < r1; r += 2) {
    process(0, r);
    if (r + 1 < r1) process(1, r + 1);
  }
  if (nv == 0) return;
  store_columns<C, V>(colpart + (grp * 3 + 0) * N + col, accb, nv);
  store_columns<C, V>(colpart + (grp * 3 + 1) * N + col, accg, nv);
  store_columns<C, V>(colpart + (grp * 3 + 2) * N + col, accz, nv);
}

// ------------------------------------------------------------------------------------------------
// B1 fused: one pass, the row held in registers (NT threads of one 16-byte vector each).  A workgroup walks rows
// blockIdx.x, blockIdx.x + gridDim.x, ... ; D rows of loads are in flight while a row is processed; one barrier
// per row (the LDS exchange slot alternates between consecutive rows).  Row data is used once per pass and is far larger
// than the caches: loads and stores of the big row-major tensors carry the non-temporal hint.
// ANY: rows start at any element and end inside a vector - the same 16-byte accesses from element-aligned addresses, the
// last, partial vector of a row element by element (one element per lane and access, as before, took 46 us for fp32
// 3001 x 1537 and 15 us for bf16).
// bf16: Phi and z phi(z) come from the LDS table, as in the forward pass's normalisation (see ActTable).
// BLK: dZ is written as [M / 32][N / 32] blocks of 32 x 32 elements, each block row-major
// (what the tuned dX and dW kernels read best, see gemm_bf16.hip).  A row's 16 bytes per lane are then 64-byte pieces,
// each half of a 128-byte line whose other half belongs to the next row: the group walks rows in neighbouring pairs,
// parks both rows' vectors in a per-wave LDS area and stores whole lines (lanes 8j .. 8j+3 the even row's piece j,
// lanes 8j+4 .. 8j+7 the odd row's).  Half-line stores straight from the registers cost the phase a third of its
// bandwidth (0.55 -> 0.73 ms on 65536 x 8192), halves merged in the L2 still a tenth.
// V: elements per thread; fewer than a vector for narrow rows (see b1_fused_impl).
// WPR: wavefronts per row.  Rows of up to 64 V or 128 V elements leave most of a workgroup's threads without one, so neighbouring
// wavefronts take rows of their own (S of them at a time) and the group's column sums meet in LDS at the end.  Whole backward
// passes with K = 8, us, one row per workgroup / so: bf16 58578 x 510 162 / 84, 65536 x 64 119 / 44, 33402 x 448 77 / 49, 20000 x 1000
// 69 / 65; fp32 65536 x 100 345 / 243, 33402 x 448 199 / 167, 30000 x 900 209 / 209.
template <class T, int NT, bool ANY, bool BLK = false, int V = 16 / (int)sizeof(T), int WPR = NT / 64>
__global__ __launch_bounds__(NT) void b1_fused_kernel(int64_t M, int64_t N, int64_t ldz, const T* __restrict__ dY,
                                                       const T* __restrict__ Z, const float* __restrict__ gamma,
                                                       const float* __restrict__ mean, const float* __restrict__ rstd,
                                                       T* __restrict__ dZ,
                                                       typename ComputeOf<T>::type* __restrict__ colpart) {
  typedef typename ComputeOf<T>::type C;
  typedef typename RawVec<T, ANY, V>::type raw_t;
  constexpr int D = 2, S = NT / 64 / WPR;
  static_assert(!BLK || (sizeof(T) == 2 && !ANY), "blocked output: bf16, whole vectors");
  __shared__ C red[2][NT / 64][2];
  __shared__ __attribute__((aligned(16))) raw_t park[BLK ? NT / 64 : 1][2][BLK ? 64 : 1];   // [wave][row of the pair][lane]
  ActTable<T, true, NT> tab;
  tab.build();
  const int slot = S == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * WPR));     // which row of the S
  const int thr = (int)threadIdx.x - slot * 64 * WPR;                                             // place in it
  const int64_t col = (int64_t)thr * V;
  const int nv = col >= N ? 0 : (N - col > V ? V : (int)(N - col));
  const int64_t left = ldz - col;              // columns of dZ this thread and those behind it write
  C accb[V], accg[V], accz[V];
  float gm[V];
#pragma unroll
  for (int v = 0; v < V; v++) { gm[v] = 0.0f; accb[v] = 0; accg[v] = 0; accz[v] = 0; }
  if (nv == V) {
#pragma unroll
    for (int v = 0; v < V; v++) gm[v] = gamma[col + v];
  } else {
#pragma unroll
    for (int v = 0; v < V; v++)
      if (v < nv) gm[v] = gamma[col + v];
  }
  // D rows are kept in flight, one per buffer; as soon as a buffer has been unpacked its refill with the row D G further
  // on is issued (G = S gridDim.x), ahead of that row's barrier and second phase.  mean and rstd travel with the row, as
  // vector loads (zero is a register the compiler cannot see through): a scalar load at the head of the row's work would
  // be waited for there.
  raw_t bdy[D], bz[D];
  float bmu[D], brs[D];
  int zero = 0;
  asm volatile("" : "+v"(zero));
  const int64_t G = (int64_t)gridDim.x * S;
  auto fetch = [&](int buf, int64_t r) {
    if (r < M) {
      bmu[buf] = mean[r + zero];
      brs[buf] = rstd[r + zero];
      if (nv > 0) {
        bdy[buf] = raw_load<T, ANY, V>(dY + r * N + col, nv);
        bz[buf] = raw_load<T, ANY, V>(Z + r * N + col, nv);
      }
    }
  };
#pragma unroll
  for (int buf = 0; buf < D; buf++)
#pragma unroll
    for (int v = 0; v < V; v++) { bdy[buf][v] = (T)0.0f; bz[buf][v] = (T)0.0f; }
  // Row-major dZ: the group walks rows b, b + G, b + 2G, ... .  Blocked dZ: rows 2b, 2b + 1, then 2G further on - the
  // two rows in flight are neighbours, so the two 64-byte halves of every line of dZ leave the same compute unit
  // within one row time and merge in its L2 (M is even where dZ is blocked).
  const int64_t lead = (int64_t)blockIdx.x * S * (BLK ? 2 : 1), first = lead + slot * (BLK ? 2 : 1);    // (lead: of slot 0)
  auto ahead = [&](int buf) -> int64_t { return BLK ? (buf >> 1) * 2 * G + (buf & 1) : buf * G; };
#pragma unroll
  for (int buf = 0; buf < D; buf++) fetch(buf, first + ahead(buf));

  const C inv_n = (C)1 / (C)N;
  auto process = [&](int buf, int64_t row) {
    const bool live = S == 1 || WPR == 1 || row < M;     // (rows that meet at barriers: past the last row all is zero, unstored)
    if (S > 1 && WPR > 1 && !live) {
      bmu[buf] = brs[buf] = 0.0f;
#pragma unroll
      for (int v = 0; v < V; v++) { bdy[buf][v] = (T)0.0f; bz[buf][v] = (T)0.0f; }
    }
    const C rs = (C)brs[buf], nmr = -(C)bmu[buf] * rs;
    C ah[V], gp[V], g[V];
    C s1 = 0, s2 = 0;
    constexpr bool kTogether = sizeof(T) == 4 && V <= 4;     // (eight elements' fp64 state at once does not fit the registers)
    C allPhi[kTogether ? V : 1], allzphi[kTogether ? V : 1];
    if constexpr (kTogether) tab.template eval<V>(bz[buf], allPhi, allzphi);
    const bool far = tab.template some_far<V>(bz[buf]);
#pragma unroll
    for (int v = 0; v < V; v++) {
      const C z = (C)to_f32<T>(bz[buf][v]);
      const C dy = (C)to_f32<T>(bdy[buf][v]);
      C Phi, zphi;
      if constexpr (kTogether) { Phi = allPhi[v]; zphi = allzphi[v]; }
      else tab.eval(z, far, Phi, zphi);
      ah[v] = (z * Phi) * rs + nmr;                        // (A - mean) rstd, one fused multiply-add
      gp[v] = (Phi + zphi) * rs;
      float gv = gm[v];
      if (sizeof(T) == 4) asm volatile("" : "+v"(gv));     // (converted here: kept as doubles they cost registers)
      g[v] = dy * (C)gv;                                   // (columns past the end: dY and gamma are zero)
      s1 += g[v];
      s2 += g[v] * ah[v];
      accb[v] += dy;
      accg[v] += dy * ah[v];
      if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
    }
    fetch(buf, row + D * G);
    if constexpr (S == 1) wg_sum2<C, NT / 64>(s1, s2, red[buf & 1]);
    else row_sum2<C, WPR>(s1, s2, red[buf & 1], slot * WPR);
    const C c1 = s1 * inv_n, c2 = s2 * inv_n;
    raw_t o;
#pragma unroll
    for (int v = 0; v < V; v++) {
      C dz = (g[v] - c1 - ah[v] * c2) * gp[v];
      if (ANY) dz = v < nv ? dz : (C)0;
      accz[v] += dz;
      o[v] = to_storage<T, C>(dz);
      if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (BLK) {
      // (every lane takes part in the stores, also one whose own columns lie past the end of the row: the pieces it
      //  stores belong to other lanes' columns)
      const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
      if (!live) return;
      if (nv > 0) park[wv][buf & 1][ln] = o;
      if (buf & 1) {
        // this wave's 16 pieces per row (piece = 4 lanes = 32 columns = one block): two stores of 8 whole lines
        const int64_t even = row - 1;
#pragma unroll
        for (int half = 0; half < 2; half++) {
          const int j = half * 8 + (ln >> 3), i = ln & 7;
          const int64_t nb = (int64_t)(wv - slot * WPR) * 16 + j;                       // block column of piece j
          if (nb * 32 < N) {                                             // N is a multiple of 32: a piece is whole or absent
            const raw_t v = park[wv][i >> 2][4 * j + (i & 3)];
            const int64_t at = (((even >> 5) * (N >> 5) + nb) << 10) + ((even & 31) << 5) + i * 8;
            __builtin_nontemporal_store(v, reinterpret_cast<raw_t*>(dZ + at));
          }
        }
      }
    } else if (live && (ANY ? left > 0 : nv > 0)) {
      raw_store<T, ANY, V>(dZ + row * ldz + col, o, nv, left);
    }
  };
  // (what ends the walk is uniform over the wavefronts that meet at a barrier)
  const int64_t back = WPR == 1 ? 0 : first - lead;
  for (int64_t row = first; row - back < M; row += D * G) {
#pragma unroll
    for (int buf = 0; buf < D; buf++)
      if (row - back + ahead(buf) < M) process(buf, row + ahead(buf));
  }
  if constexpr (S > 1) {
    // the slots' sums meet in slot 0
    __shared__ C comb[3 * V][(S - 1) * 64 * WPR];
    if (slot > 0) {
      const int at = (int)threadIdx.x - 64 * WPR;
#pragma unroll
      for (int v = 0; v < V; v++) { comb[v][at] = accb[v]; comb[V + v][at] = accg[v]; comb[2 * V + v][at] = accz[v]; }
    }
    __syncthreads();
    if (slot > 0) return;
#pragma unroll
    for (int w = 0; w < S - 1; w++)
#pragma unroll
      for (int v = 0; v < V; v++) {
        accb[v] += comb[v][w * 64 * WPR + thr];
        accg[v] += comb[V + v][w * 64 * WPR + thr];
        accz[v] += comb[2 * V + v][w * 64 * WPR + thr];
      }
  }
  if (nv > 0) {
    store_columns<C, V>(colpart + ((int64_t)blockIdx.x * 3 + 0) * N + col, accb, nv);
    store_columns<C, V>(colpart + ((int64_t)blockIdx.x * 3 + 1) * N + col, accg, nv);
    store_columns<C, V>(colpart + ((int64_t)blockIdx.x * 3 + 2) * N + col, accz, nv);
  }
}

// ------------------------------------------------------------------------------------------------
// B2: colpart [groups][3][N] -> dbeta, dgamma, db (b2_columns) in a launch of its own (bf16 storage; the fp32 path ends
// with f64_finish_kernel).
__global__ __launch_bounds__(1024) void b2_kernel(int64_t N, int groups, const float* __restrict__ colpart,
                                                  float* __restrict__ dbeta, float* __restrict__ dgamma,
                                                  float* __restrict__ db) {
  __shared__ double red[16][64];
  const int which = blockIdx.y;
  b2_columns<float>(N, groups, (int)gridDim.y, colpart, (int)blockIdx.x, which,
                    which == 0 ? dbeta : (which == 1 ? dgamma : db), red);
}

// The tail of a bf16 backward pass in one launch, for shapes where the contractions leave split reductions behind:
// workgroups [0, a.blocks) and [a.blocks, a.blocks + b.blocks) add the fp32 partial products of up to two outputs
// (4096 elements per workgroup, partials summed in index order, one rounding to bf16), the remaining kinds ceil(N / 64)
// workgroups finish the column sums exactly as b2_kernel does.  Small dependent launches cost a few microseconds each
// whatever they do, which is what this saves for mid-sized layers.
__global__ __launch_bounds__(1024) void finish_kernel(TailSums j) {
  __shared__ double red[16][64];
  int id = (int)blockIdx.x;
  for (int k = 0; k < 2; k++) {
    if (id < j.blocks[k]) {
      const int64_t i = ((int64_t)id * 1024 + threadIdx.x) * 4;
      if (i >= j.n[k]) return;
      const float* part = j.part[k];
      f32x4 acc = *reinterpret_cast<const f32x4*>(part + i);
      int q = 1;
      for (; q + 4 <= j.parts[k]; q += 4) {        // (four loads in flight)
        f32x4 t[4];
#pragma unroll
        for (int u = 0; u < 4; u++) t[u] = *reinterpret_cast<const f32x4*>(part + (int64_t)(q + u) * j.stride[k] + i);
#pragma unroll
        for (int u = 0; u < 4; u++) { acc[0] += t[u][0]; acc[1] += t[u][1]; acc[2] += t[u][2]; acc[3] += t[u][3]; }
      }
      for (; q < j.parts[k]; q++) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(part + (int64_t)q * j.stride[k] + i);
        acc[0] += t[0]; acc[1] += t[1]; acc[2] += t[2]; acc[3] += t[3];
      }
      bf16x4 o;
      o[0] = (bf16_t)acc[0]; o[1] = (bf16_t)acc[1]; o[2] = (bf16_t)acc[2]; o[3] = (bf16_t)acc[3];
      bf16_t* out = static_cast<bf16_t*>(j.out[k]) + i;
      if (i + 4 <= j.n[k]) {
        *reinterpret_cast<bf16x4*>(out) = o;
      } else {
        for (int e = 0; i + e < j.n[k]; e++) out[e] = o[e];
      }
      return;
    }
    id -= j.blocks[k];
  }
  const int cblocks = (int)((j.N + 63) / 64);
  const int which = id / cblocks;
  b2_columns<float>(j.N, j.groups, j.kinds, j.colpart, id % cblocks, which,
                    which == 0 ? j.col_out[0] : (which == 1 ? j.col_out[1] : j.col_out[2]), red);
}


// ------------------------------------------------------------------------------------------------
// Normalisation with its own statistics, fp32 storage: a workgroup of NT threads owns a row and holds it in registers
// over the three sweeps (activation and sum; deviations and their squares; scale, shift, store), S vectors of four per
// thread, so that a row is read once.  ACT as above; Z and Y may be the same buffer (a thread reads its part of a row
// before it writes it).
// Bound: HBM (with GELU: fp64 arithmetic).  What keeps loads in flight: the next row's vectors are fetched as soon as this
// one's are unpacked, ahead of its two reductions, and several workgroups share a compute unit.  The row streams past the
// caches: LayerNorm of 8192 x 4096 took 74 us with three trips through memory and caches per row, 64 us in this form with
// plain loads and stores, 52 us (5.2 TB/s) with the non-temporal hint on both.
// Rows start at any element: the vectors are read and written with the widest instructions from element-aligned
// addresses (the hardware splits what straddles a line), the last, partial one of a row element by element.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

// PARTS: Z is not there yet - its tiles' parts (gemm_f64.hip, all of them split) are added here in order, with the bias, rounded
// and written, to the same bits as by the launch that would do it in between (whole forward passes, us, with that / so: 256^3 14.6 /
// 12.0, 33 x 1000 x 70 16.5 / 12.2, 128 x 4096 x 1024 34.0 / 30.4, 512^3 19.9 / 17.7, 1000 x 700 x 1000 39.2 / 38.9).
template <int NT, int S, int ACT, bool PARTS = false>
__global__ __launch_bounds__(NT) void row_wg_kernel(int64_t M, int64_t N, float eps, const float* Z,
                                                    const float* __restrict__ gamma, const float* __restrict__ beta,
                                                    float* Y, float* __restrict__ mean, float* __restrict__ rstd, F64Sums q) {
  typedef ActTable<float, false, NT> Act;
  constexpr int V = 4, NW = NT / 64;
  constexpr bool kKeep = NT < 1024;      // gamma and beta stay in registers (1024 threads have 128 each: read per row)
  __shared__ double red[2][NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int col[S], nv[S];
  float gm[S][V], bt[S][V];
  auto affine = [&](int s) {
    if (nv[s] == V) {
      const f32x4 g4 = *reinterpret_cast<const f32x4*>(gamma + col[s]);
      const f32x4 b4 = *reinterpret_cast<const f32x4*>((ACT == ACT_RMS ? gamma : beta) + col[s]);
#pragma unroll
      for (int v = 0; v < V; v++) { gm[s][v] = g4[v]; bt[s][v] = ACT == ACT_RMS ? 0.0f : b4[v]; }
    } else {
#pragma unroll
      for (int v = 0; v < V; v++) {
        gm[s][v] = v < nv[s] ? gamma[col[s] + v] : 0.0f;
        bt[s][v] = (ACT != ACT_RMS && v < nv[s]) ? beta[col[s] + v] : 0.0f;
      }
    }
  };
#pragma unroll
  for (int s = 0; s < S; s++) {
    col[s] = (s * NT + (int)threadIdx.x) * V;
    const int64_t left = N - col[s];
    nv[s] = left < 0 ? 0 : (left > V ? V : (int)left);
    if (kKeep) affine(s);
  }
  f32x4_u raw[S];
  auto fetch = [&](int64_t row) {
    if constexpr (PARTS) {
      if (row >= M) return;
#pragma unroll
      for (int s = 0; s < S; s++) {
        // (four columns from a multiple of four on lie in one tile)
        const double* p = q.part + ((row >> 6) * q.tiles_j + (col[s] >> 6)) * 4096 + (row & 63) * 64 + (col[s] & 63);
        f64x4 z = {0.0, 0.0, 0.0, 0.0};
        if (nv[s] > 0) {
          z = *reinterpret_cast<const f64x4*>(p);
#pragma unroll 4
          for (int k = 1; k < q.split; k++) {
            const f64x4 x = *reinterpret_cast<const f64x4*>(p + (int64_t)k * q.stride);
#pragma unroll
            for (int v = 0; v < V; v++) z[v] += x[v];
          }
        }
#pragma unroll
        for (int v = 0; v < V; v++) {
          raw[s][v] = v < nv[s] ? (float)(z[v] + (double)q.bias[col[s] + v]) : 0.0f;
          if (v < nv[s] && q.Z != Y) q.Z[row * N + col[s] + v] = raw[s][v];     // (inference keeps no Z: it would lie in Y)
        }
      }
      return;
    }
    const float* z = Z + (row < M ? row : M - 1) * N;  // past the last row: a harmless re-read of it
#pragma unroll
    for (int s = 0; s < S; s++) {
      if (nv[s] == V) {
        raw[s] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_u*>(z + col[s]));
      } else {
#pragma unroll
        for (int v = 0; v < V; v++) raw[s][v] = v < nv[s] ? z[col[s] + v] : 0.0f;
      }
    }
  };
  // sum over the workgroup; consecutive calls use the two slots in turn, so one barrier each is enough: a slot is
  // written again only after the barrier of the call in between
  int slot = 0;
  auto wg_sum = [&](double x) -> double {
    x = wave_sum(x);
    if constexpr (NW == 1) {
      return x;
    } else {
      if (lane == 0) red[slot][wave] = x;
      __syncthreads();
      double t = red[slot][0];
#pragma unroll
      for (int w = 1; w < NW; w++) t += red[slot][w];
      slot ^= 1;
      return t;
    }
  };
  const double inv_n = 1.0 / (double)N;
  fetch(blockIdx.x);
  Act act;
  if (ACT == ACT_GELU) act.build();
  for (int64_t row = blockIdx.x; row < M; row += gridDim.x) {
    double a[S][V], sum = 0;
#pragma unroll
    for (int s = 0; s < S; s++) {
#pragma unroll
      for (int v = 0; v < V; v++) a[s][v] = 0;
      if (nv[s] == 0) continue;                        // (a whole wavefront past the end of the row skips the activation)
      if constexpr (ACT == ACT_GELU) act.template gelu<V>(raw[s], a[s]);     // zeros past the end of the row: GELU(0) = 0
#pragma unroll
      for (int v = 0; v < V; v++) {
        const double z = (double)raw[s][v];
        if (ACT != ACT_GELU) a[s][v] = z;
        sum += ACT == ACT_RMS ? z * z : a[s][v];
      }
    }
    fetch(row + gridDim.x);
    double rs;
    if (ACT == ACT_RMS) {
      rs = 1.0 / sqrt(wg_sum(sum) * inv_n + (double)eps);
    } else {
      const double mu = wg_sum(sum) * inv_n;
      double m2 = 0;
#pragma unroll
      for (int s = 0; s < S; s++)
#pragma unroll
        for (int v = 0; v < V; v++) {
          a[s][v] = v < nv[s] ? a[s][v] - mu : 0.0;
          m2 += a[s][v] * a[s][v];
        }
      rs = 1.0 / sqrt(wg_sum(m2) * inv_n + (double)eps);
      if (threadIdx.x == 0) { mean[row] = (float)mu; rstd[row] = (float)rs; }
    }
    float* y = Y + row * N;
#pragma unroll
    for (int s = 0; s < S; s++) {
      if (!kKeep) affine(s);
      f32x4_u o;
#pragma unroll
      for (int v = 0; v < V; v++) o[v] = (float)(a[s][v] * rs * (double)gm[s][v] + (double)bt[s][v]);
      if (nv[s] == V) {
        __builtin_nontemporal_store(o, reinterpret_cast<f32x4_u*>(y + col[s]));
      } else {
#pragma unroll
        for (int v = 0; v < V; v++)
          if (v < nv[s]) y[col[s] + v] = o[v];
      }
    }
  }
}

// F2 for narrow rows (up to 16 K elements): sixteen lanes share a row, lane l holding its elements l, l + 16, ..., so that a
// wavefront has four rows at once, whatever their alignment.  Bound: the latency of a row's chain of loads and sums (a wavefront
// per row, or a workgroup of fp32 storage, has a few lanes' work in it): inference, us, 60000 x 24 x 15 fp32 69 -> 19, bf16
// 20000 x 16 x 15 22.5 -> 7.5, 60000 x 99 x 127 67 -> 34.
template <class T, int K>
__global__ __launch_bounds__(256) void f2_narrow_kernel(int64_t M, int64_t N, float eps, const T* Z, const float* __restrict__ gamma,
                                                        const float* __restrict__ beta, T* Y, float* __restrict__ mean,
                                                        float* __restrict__ rstd) {
  typedef typename ComputeOf<T>::type C;
  ActTable<T, false, 256> tab;
  tab.build();
  const int l = threadIdx.x & 15;
  float gm[K], bt[K];
  int at[K];
#pragma unroll
  for (int k = 0; k < K; k++) {
    at[k] = l + 16 * k < N ? l + 16 * k : (int)N - 1;              // past the end: the last element again, unused
    gm[k] = gamma[at[k]];
    bt[k] = beta[at[k]];
  }
  const double inv_n = 1.0 / (double)N;
  const int64_t step = (int64_t)gridDim.x * 16;
  T raw[K];
  auto fetch = [&](int64_t row) {
    const T* z = Z + (row < M ? row : M - 1) * N;
#pragma unroll
    for (int k = 0; k < K; k++) raw[k] = z[at[k]];
  };
  // (the lanes of a wavefront stay together: row16_sum; a row past the last is done like it and not stored)
  int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  fetch(row);
  for (int64_t lead = (int64_t)blockIdx.x * 16; lead < M; lead += step, row += step) {
    C a[K], sum = 0, sq = 0;
    if constexpr (sizeof(T) == 4) tab.template gelu<K>(raw, a);
#pragma unroll
    for (int k = 0; k < K; k++) {
      if constexpr (sizeof(T) == 2) a[k] = l + 16 * k < N ? tab.gelu(to_f32<T>(raw[k])) : 0.0f;
      else a[k] = l + 16 * k < N ? a[k] : 0.0;
      sum += a[k];
    }
    fetch(row + step);
    const double mu = (double)row16_sum(sum) * inv_n;
    const C m = (C)mu;
#pragma unroll
    for (int k = 0; k < K; k++) {
      a[k] = l + 16 * k < N ? a[k] - m : (C)0;
      sq += a[k] * a[k];
    }
    const double var = (double)row16_sum(sq) * inv_n + (double)eps;
    C rs;
    if constexpr (sizeof(T) == 4) rs = 1.0 / sqrt(var);
    else rs = inv_sqrt(var);
    if (row < M) {
      if (l == 0) { mean[row] = (float)mu; rstd[row] = (float)rs; }
#pragma unroll
      for (int k = 0; k < K; k++)
        if (l + 16 * k < N) Y[row * N + l + 16 * k] = to_storage<T, C>(a[k] * rs * (C)gm[k] + (C)bt[k]);
    }
  }
}

// F2 for rows too long for the registers of a workgroup: two launches over segments of kLongVectors vectors per thread.  The
// first leaves every segment's mean and sum of squared deviations (fp64) in `part` [M][segments], the second merges a row's
// and normalises its segment.  So GELU is evaluated twice per element and the row read twice, and a few long rows fill the
// chip: a workgroup takes rows_per_wg rows of one segment (gamma and beta stay in its registers), as many as leave about 2048
// workgroups.
// Bound: HBM for bf16, fp64 arithmetic for fp32 storage.  One workgroup per row that streams it three times took, whole
// inference calls, us, that / now: fp32 17 x 42 x 24886 141 / 19, 256 x 34 x 44889 343 / 122; bf16 32 x 256 x 78860 236 / 34,
// 4096 x 256 x 65536 686 / 606; an earlier form with the sums in the contraction's epilogue, which read each row once, 43, 153, 86
// and 612.
constexpr int kLongVectors = 2;
template <class T> constexpr int64_t long_segment() { return 256 * (16 / (int)sizeof(T)) * kLongVectors; }

// One thread's vectors of a segment: columns, how many elements each has, and the raw values of two rows in flight
template <class T, bool ANY> struct LongLane {
  static constexpr int V = 16 / (int)sizeof(T);
  int64_t col[kLongVectors];
  int nv[kLongVectors];
  typename RawVec<T, ANY>::type raw[2][kLongVectors];
  __device__ __forceinline__ void init(int64_t N, int64_t c0) {
#pragma unroll
    for (int s = 0; s < kLongVectors; s++) {
      col[s] = c0 + (s * 256 + (int)threadIdx.x) * V;
      const int64_t left = N - col[s];
      nv[s] = left <= 0 ? 0 : (left > V ? V : (int)left);
#pragma unroll
      for (int v = 0; v < V; v++) raw[0][s][v] = raw[1][s][v] = (T)0.0f;
    }
  }
  __device__ __forceinline__ void fetch(int buf, const T* Z, int64_t N, int64_t row, int64_t end) {
    if (row >= end) return;
#pragma unroll
    for (int s = 0; s < kLongVectors; s++)
      if (nv[s] > 0) raw[buf][s] = row_load<T, ANY>(Z + row * N + col[s], nv[s]);
  }
};

// A wavefront's sums are of the differences to its first element: both in one pass, and nothing cancels where the elements
// are nearly equal.  The four wavefronts' means and sums of squares are then merged.
template <class T, bool ANY>
__global__ __launch_bounds__(256) void long_moments_kernel(int64_t M, int64_t N, int segments, int rows_per_wg, const T* Z,
                                                           double2* __restrict__ part) {
  typedef typename ComputeOf<T>::type C;
  constexpr int V = LongLane<T, ANY>::V;
  __shared__ double red[2][2][4][2];
  ActTable<T, false, 256> tab;
  tab.build();
  const int seg = blockIdx.x % segments, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = (int64_t)(blockIdx.x / segments) * rows_per_wg, r1 = r0 + rows_per_wg < M ? r0 + rows_per_wg : M;
  LongLane<T, ANY> l;
  l.init(N, seg * long_segment<T>());
  double count[4], n = 0.0;                    // elements of each wavefront, and of the segment
#pragma unroll
  for (int w = 0; w < 4; w++) {
    int64_t c = 0;
#pragma unroll
    for (int s = 0; s < kLongVectors; s++) {
      const int64_t left = N - (seg * long_segment<T>() + (s * 256 + w * 64) * V);
      c += left <= 0 ? 0 : (left > 64 * V ? 64 * V : left);
    }
    count[w] = (double)c;
    n += count[w];
  }
  const double inv_n = 1.0 / n, n_wave = count[wave], inv_wave = n_wave > 0.0 ? 1.0 / n_wave : 0.0;
  l.fetch(0, Z, N, r0, r1);
  l.fetch(1, Z, N, r0 + 1, r1);
  // two rows at a time: their reductions overlap and share a barrier
  for (int64_t row = r0; row < r1; row += 2) {
    const int slot = row_sum_slot(1, (int)((row - r0) >> 1), 0);
    double sum[2], sq[2];
    C base[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
      sum[k] = 0.0; sq[k] = 0.0; base[k] = 0;
      if (k > 0 && row + k >= r1) continue;                      // (uniform)
      C a[kLongVectors][V];
#pragma unroll
      for (int s = 0; s < kLongVectors; s++) tab.template gelu<V>(l.raw[k][s], a[s]);
      l.fetch(k, Z, N, row + k + 2, r1);
      base[k] = read_lane(a[0][0], 0);
#pragma unroll
      for (int s = 0; s < kLongVectors; s++) {
        if (l.nv[s] == 0) continue;
        C ps = 0, pq = 0;
#pragma unroll
        for (int v = 0; v < V; v++) {
          const C d = !ANY || v < l.nv[s] ? a[s][v] - base[k] : (C)0;
          ps += d;
          pq = __builtin_elementwise_fma(d, d, pq);
        }
        sum[k] += (double)ps;
        sq[k] += (double)pq;
      }
    }
#pragma unroll
    for (int k = 0; k < 2; k++) { sum[k] = wave_sum(sum[k]); sq[k] = wave_sum(sq[k]); }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int k = 0; k < 2; k++) {
        red[slot][k][wave][0] = (double)base[k] + sum[k] * inv_wave;
        red[slot][k][wave][1] = sq[k] - sum[k] * sum[k] * inv_wave;
      }
    }
    __syncthreads();
    if (threadIdx.x < 2 && row + threadIdx.x < r1) {
      const double (*q)[2] = red[slot][threadIdx.x];
      double mean = 0.0, m2 = 0.0;
#pragma unroll
      for (int w = 0; w < 4; w++) mean += count[w] * q[w][0];
      mean *= inv_n;
#pragma unroll
      for (int w = 0; w < 4; w++) { const double d = q[w][0] - mean; m2 += q[w][1] + count[w] * d * d; }
      part[(row + threadIdx.x) * segments + seg] = double2{mean, m2};
    }
  }
}

template <class T, bool ANY>
__global__ __launch_bounds__(256) void long_apply_kernel(int64_t M, int64_t N, int segments, int rows_per_wg, float eps,
                                                         const T* Z, const double2* __restrict__ part,
                                                         const float* __restrict__ gamma, const float* __restrict__ beta, T* Y,
                                                         float* __restrict__ mean_out, float* __restrict__ rstd_out) {
  typedef typename ComputeOf<T>::type C;
  constexpr int V = LongLane<T, ANY>::V;
  __shared__ C stats[2][16][2];                // mean and rstd of sixteen rows, twice
  ActTable<T, false, 256> tab;
  tab.build();
  const int seg = blockIdx.x % segments;
  const int64_t r0 = (int64_t)(blockIdx.x / segments) * rows_per_wg, r1 = r0 + rows_per_wg < M ? r0 + rows_per_wg : M;
  LongLane<T, ANY> l;
  l.init(N, seg * long_segment<T>());
  float gm[kLongVectors][V], bt[kLongVectors][V];
#pragma unroll
  for (int s = 0; s < kLongVectors; s++) {
    if (l.nv[s] == V) {
#pragma unroll
      for (int v = 0; v < V; v += 4) {
        const f32x4 g4 = *reinterpret_cast<const f32x4*>(gamma + l.col[s] + v), b4 = *reinterpret_cast<const f32x4*>(beta + l.col[s] + v);
#pragma unroll
        for (int e = 0; e < 4; e++) { gm[s][v + e] = g4[e]; bt[s][v + e] = b4[e]; }
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; v++) {
        gm[s][v] = v < l.nv[s] ? gamma[l.col[s] + v] : 0.0f;
        bt[s][v] = v < l.nv[s] ? beta[l.col[s] + v] : 0.0f;
      }
    }
  }
  const double full = (double)long_segment<T>(), last = (double)(N - (segments - 1) * long_segment<T>());
  auto process = [&](int buf, int64_t row) {
    const int at = (int)(row - r0) & 15, half = (int)((row - r0) >> 4) & 1;
    const C mu = stats[half][at][0], rs = stats[half][at][1];
    typename RawVec<T, ANY>::type o[kLongVectors];
#pragma unroll
    for (int s = 0; s < kLongVectors; s++) {
      C a[V];
      tab.template gelu<V>(l.raw[buf][s], a);
#pragma unroll
      for (int v = 0; v < V; v++) o[s][v] = to_storage<T, C>((a[v] - mu) * rs * (C)gm[s][v] + (C)bt[s][v]);
    }
    l.fetch(buf, Z, N, row + 2, r1);
#pragma unroll
    for (int s = 0; s < kLongVectors; s++)
      if (l.nv[s] > 0) raw_store<T, ANY>(Y + row * N + l.col[s], o[s], l.nv[s], l.nv[s]);
  };
  l.fetch(0, Z, N, r0, r1);
  l.fetch(1, Z, N, r0 + 1, r1);
  for (int64_t row = r0; row < r1; row += 2) {
    if (((row - r0) & 15) == 0) {
      // the next sixteen rows' segments merged, sixteen lanes per row (the half written was read before the last barrier)
      const int t0 = threadIdx.x & 15;
      const int64_t q = row + (threadIdx.x >> 4);
      const double2* p = part + (q < M ? q : M - 1) * segments;
      double mean = 0.0, m2 = 0.0;
      for (int t = t0; t < segments; t += 16) mean += (t == segments - 1 ? last : full) * p[t].x;
      mean = row16_sum(mean) / (double)N;
      for (int t = t0; t < segments; t += 16) {
        const double d = p[t].x - mean;
        m2 += p[t].y + (t == segments - 1 ? last : full) * d * d;
      }
      const double rstd = 1.0 / sqrt(row16_sum(m2) / (double)N + (double)eps);
      if (t0 == 0) {
        C* out = stats[(int)((row - r0) >> 4) & 1][threadIdx.x >> 4];
        out[0] = (C)mean; out[1] = (C)rstd;
        if (seg == 0 && q < r1) { mean_out[q] = (float)mean; rstd_out[q] = (float)rstd; }
      }
      __syncthreads();
    }
    process(0, row);
    if (row + 1 < r1) process(1, row + 1);
  }
}

// The stand-alone norms, which have no scratch, for rows that long: the row is read from memory (and then from the caches)
// once per sweep, as in the paper's two-step LayerNorm and strided RMSNorm kernels.
template <class T, int V, int ACT>
__global__ __launch_bounds__(256) void row_stream_kernel(int64_t M, int64_t N, float eps, const T* __restrict__ A,
                                                         const float* __restrict__ gamma, const float* __restrict__ beta,
                                                         T* __restrict__ Y, float* __restrict__ mean,
                                                         float* __restrict__ rstd) {
  typedef typename ComputeOf<T>::type C;
  __shared__ C red[2][4][2];
  for (int64_t row = blockIdx.x; row < M; row += gridDim.x) {
    const T* a = A + row * N;
    C s1 = 0, s2 = 0;
    for (int64_t col = (int64_t)threadIdx.x * V; col < N; col += 256 * V) {
      C x[V];
      VecIO<T, V>::load(a + col, x);
#pragma unroll
      for (int v = 0; v < V; v++) { s1 += x[v]; s2 += x[v] * x[v]; }
    }
    wg_sum2<C, 4>(s1, s2, red[0]);
    C mu = 0, rs;
    if (ACT == ACT_RMS) {
      rs = (C)1 / sqrt(s2 / (C)N + (C)eps);
    } else {
      mu = s1 / (C)N;
      C d2 = 0, dummy = 0;
      for (int64_t col = (int64_t)threadIdx.x * V; col < N; col += 256 * V) {
        C x[V];
        VecIO<T, V>::load(a + col, x);
#pragma unroll
        for (int v = 0; v < V; v++) { const C d = x[v] - mu; d2 += d * d; }
      }
      wg_sum2<C, 4>(d2, dummy, red[1]);
      rs = (C)1 / sqrt(d2 / (C)N + (C)eps);
      if (threadIdx.x == 0) { mean[row] = (float)mu; rstd[row] = (float)rs; }
    }
    for (int64_t col = (int64_t)threadIdx.x * V; col < N; col += 256 * V) {
      C x[V], y[V];
      VecIO<T, V>::load(a + col, x);
#pragma unroll
      for (int v = 0; v < V; v++) {
        if (ACT == ACT_RMS) y[v] = x[v] * rs * (C)gamma[col + v];
        else y[v] = (x[v] - mu) * rs * (C)gamma[col + v] + (C)beta[col + v];
      }
      VecIO<T, V>::store(Y + row * N + col, y);
    }
    __syncthreads();   // the exchange slots are reused by the next row
  }
}

// Column sums of a row-major matrix, first stage: workgroup g sums rows g, g + G, ... of a strip of 256 V columns
// into colpart[g][N] (arithmetic type); b2_kernel finishes them.  Coalesced along the row, no atomics.
// BLK: the matrix is stored in 32 x 32 blocks (see gemm_bf16.hip); a lane's 16 bytes are then a quarter of a 64-byte
// piece, and the group walks rows in neighbouring pairs, whose pieces share a line (M even).
template <class T, int V, bool BLK = false>
__global__ __launch_bounds__(256) void colsum_partial_kernel(int64_t M, int64_t N, int64_t ldg, int strips, int groups,
                                                             const T* __restrict__ G,
                                                             typename ComputeOf<T>::type* __restrict__ colpart) {
  typedef typename ComputeOf<T>::type C;
  const int strip = blockIdx.x % strips;
  const int grp = blockIdx.x / strips;
  const int64_t col = ((int64_t)strip * 256 + threadIdx.x) * V;
  if (col >= N) return;
  C acc[V];
#pragma unroll
  for (int v = 0; v < V; v++) acc[v] = 0;
  if constexpr (BLK) {
    const int64_t cb = ((col >> 5) << 10) + (col & 31);
#pragma unroll 2
    for (int64_t r = 2 * (int64_t)grp; r < M; r += 2 * (int64_t)groups) {
      const T* base = G + (((r >> 5) * (N >> 5)) << 10) + ((r & 31) << 5) + cb;
      C x[V], y[V];
      VecIO<T, V>::load(base, x);
      VecIO<T, V>::load(base + 32, y);     // row r + 1 (r is even: same block row)
#pragma unroll
      for (int v = 0; v < V; v++) acc[v] += x[v] + y[v];
    }
  } else {
#pragma unroll 4
    for (int64_t r = grp; r < M; r += groups) {
      C x[V];
      VecIO<T, V>::load(G + r * ldg + col, x);
#pragma unroll
      for (int v = 0; v < V; v++) acc[v] += x[v];
    }
  }
  if constexpr (V > 1) store_columns<C, V>(colpart + (int64_t)grp * N + col, acc, N - col > V ? V : (int)(N - col));
  else colpart[(int64_t)grp * N + col] = acc[0];
}

// H = SiLU(G) * U, element by element (the gated feed-forward block's activation); H may be G or U.
template <class T, int V>
__global__ __launch_bounds__(256) void silu_mul_kernel(int64_t n, const T* G, const T* U, T* H) {
  typedef typename ComputeOf<T>::type C;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V; i < n; i += (int64_t)gridDim.x * 256 * V) {
    C g[V], u[V], h[V];
    VecIO<T, V>::load(G + i, g);
    VecIO<T, V>::load(U + i, u);
#pragma unroll
    for (int v = 0; v < V; v++) {
      if constexpr (sizeof(C) == 8) h[v] = g[v] / (1.0 + exp(-g[v])) * u[v];
      else h[v] = g[v] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * g[v])) * u[v];
    }
    VecIO<T, V>::store(H + i, h);
  }
}

template <class T> void b1a_impl(int64_t M, int64_t N, const void* dY, const void* Z, const float* gamma,
                                 const float* mean, const float* rstd, void* c12, hipStream_t s) {
  typedef typename ComputeOf<T>::type C;
  const unsigned blocks = (unsigned)(M < 4096 ? M : 4096);
  auto kern = N % (16 / (int)sizeof(T)) == 0 ? b1a_kernel<T, false> : b1a_kernel<T, true>;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, s, M, N, (const T*)dY, (const T*)Z, gamma, mean, rstd, (C*)c12);
}

template <class T> void b1b_impl(int64_t M, int64_t N, int64_t ldz, int rows_per_group, int groups, const void* dY, const void* Z,
                                 const float* gamma, const float* mean, const float* rstd, const void* c12, void* dZ,
                                 void* colpart, hipStream_t s) {
  typedef typename ComputeOf<T>::type C;
  constexpr int V = 16 / (int)sizeof(T);
  const int strips = (int)((N + 256 * (int64_t)V - 1) / (256 * (int64_t)V));
  const int64_t blocks = (int64_t)strips * groups;
  auto kern = N % V == 0 && ldz % V == 0 ? b1b_kernel<T, false> : b1b_kernel<T, true>;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, M, N, ldz, rows_per_group, strips, (const T*)dY,
                     (const T*)Z, gamma, mean, rstd, (const C*)c12, (T*)dZ, (C*)colpart);
}

// Threads of a workgroup of the fused kernel: one 16-byte vector each, the row's pitch in dZ included (the surplus columns
// of a padded dZ are zeroed by the threads behind the row's end).  0: the row does not fit.
inline int fused_threads(int dt, int64_t N, int64_t ldz) {
  const int V = dt == kF32 ? 4 : 8;
  const int64_t per_row = ((ldz > N ? ldz : N) + V - 1) / V;
  if (per_row <= 256) return 256;
  if (per_row <= 512) return 512;
  return per_row <= 1024 ? 1024 : 0;
}

// Rows that a workgroup of the fused kernel has in hand at once: narrow rows are a wavefront's (64 vectors) or two's.
inline int b1_slots(int dt, int64_t N, int64_t ldz) {
  const int V = dt == kF32 ? 4 : 8;
  const int64_t per_row = ((ldz > N ? ldz : N) + V - 1) / V;
  return per_row <= 64 ? 4 : (per_row <= 128 ? 2 : 1);
}

template <class T> void b1_fused_impl(int64_t M, int64_t N, int64_t ldz, int groups, bool blocked, const void* dY, const void* Z,
                                      const float* gamma, const float* mean, const float* rstd, void* dZ,
                                      void* colpart, hipStream_t s) {
  typedef typename ComputeOf<T>::type C;
  constexpr int V = 16 / (int)sizeof(T);
  const int nt = fused_threads(sizeof(T) == 4 ? kF32 : kBF16, N, ldz);   // callers check b1_fused_supported first
  // a row of whole vectors, or one that starts or ends inside a vector or is followed by columns to be zeroed
  const bool any = N % V != 0 || ldz != N;
  const dim3 grid((unsigned)groups);
#define FDL_B1_ARGS s, M, N, ldz, (const T*)dY, (const T*)Z, gamma, mean, rstd, (T*)dZ, (C*)colpart
  if constexpr (sizeof(T) == 4) {
    // (1024 threads have 128 registers each, too few for the fp64 state of four columns: 8192 x 4096 221 us, half as many threads
    // of eight 123; at up to 2048 columns 256 threads of eight lose to 512 of four, 34 to 25 for 3001 x 1537)
    if (nt == 1024) {
      if (N % 8 != 0 || ldz != N) hipLaunchKernelGGL((b1_fused_kernel<T, 512, true, false, 8>), grid, dim3(512), 0, FDL_B1_ARGS);
      else hipLaunchKernelGGL((b1_fused_kernel<T, 512, false, false, 8>), grid, dim3(512), 0, FDL_B1_ARGS);
      return;
    }
  }
#define FDL_B1F(NT, ANY, BLK) hipLaunchKernelGGL((b1_fused_kernel<T, NT, ANY, BLK>), grid, dim3(NT), 0, FDL_B1_ARGS)
#define FDL_B1F_NT(ANY, BLK)                                                                                              \
  do {                                                                                                                    \
    if (nt == 256) FDL_B1F(256, ANY, BLK);                                                                                \
    else if (nt == 512) FDL_B1F(512, ANY, BLK);                                                                           \
    else if constexpr (sizeof(T) == 2) FDL_B1F(1024, ANY, BLK);                                                           \
  } while (0)
  // narrow rows: a wavefront or two per row, an element, four or a vector per thread (b1_slots says how many rows a group takes)
#define FDL_B1N(ANY, BLK, VV, WPR) hipLaunchKernelGGL((b1_fused_kernel<T, 256, ANY, BLK, VV, WPR>), grid, dim3(256), 0, FDL_B1_ARGS)
  const int slots = b1_slots(sizeof(T) == 4 ? kF32 : kBF16, N, ldz);
  if constexpr (sizeof(T) == 2) {
    if (blocked) {
      if (slots == 4) FDL_B1N(false, true, V, 1); else if (slots == 2) FDL_B1N(false, true, V, 2); else FDL_B1F_NT(false, true);
      return;
    }
    if (slots == 4 && ldz <= 256 && ldz > 64) {
      if (N % 4 != 0 || ldz != N) FDL_B1N(true, false, 4, 1); else FDL_B1N(false, false, 4, 1);
      return;
    }
  }
  if (slots == 4) {
    if (ldz <= 64) FDL_B1N(true, false, 1, 1); else if (any) FDL_B1N(true, false, V, 1); else FDL_B1N(false, false, V, 1);
    return;
  }
  if (slots == 2) {
    if (any) FDL_B1N(true, false, V, 2); else FDL_B1N(false, false, V, 2);
    return;
  }
#undef FDL_B1N
  if (any) FDL_B1F_NT(true, false);
  else FDL_B1F_NT(false, false);
#undef FDL_B1F_NT
#undef FDL_B1F
#undef FDL_B1_ARGS
}

}  // namespace

// one instantiation: gamma/beta (4 KB per 512 columns) plus the Phi table can exceed the default 64 KB of dynamic LDS
template <int CH, int FIT, int NT, int ACT, int WPR = 1>
void launch_f2_rows_one(int64_t wgs, int stretches, hipStream_t s, int64_t M, int64_t N, float eps, const bf16_t* Z, const float* gamma,
                        const float* beta, bf16_t* Y, float* mean, float* rstd) {
  constexpr size_t kLds = (affine_in_lds(CH * WPR) ? (size_t)CH * WPR * 4096 : 0) + (ACT == ACT_GELU ? GaussTable<false>::kBytes : 0);
  auto kern = f2_rows_kernel<CH, FIT, NT, ACT, WPR>;
  if constexpr (kLds > 64 * 1024) {
    static OnceFlags configured;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)kLds, &configured)) return;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(NT), kLds, s, M, N, eps, Z, gamma, beta, Y, mean, rstd, stretches);
}

constexpr int64_t kMemorySideCache = (int64_t)256 << 20;      // bytes
template <int ACT>
void launch_rows_act(int64_t M, int64_t N, float eps, const void* Zsave, const float* gamma, const float* beta, void* Y,
                     float* mean, float* rstd, hipStream_t s) {
  // Rows of 16384 take 16 vectors per lane.  The others, whose masks cost registers (one wavefront per SIMD with
  // 16 vectors), take at most 8 and more wavefronts per row: 10000 x 5000 70.7 -> 50.1 us, 8192 x 10496 101.6 -> 71.6,
  // 3001 x 12345 64.9 -> 48.6.
  // Rows of up to 512 columns are one vector per lane (as half of two, us: LayerNorm 65536 x 100 28.8 -> 21.0, 25535 x 337 16.4 -> 12.5,
  // 58578 x 510 31.7 -> 25.0; forward pass of 65536 x 64 x 256 44 -> 36.5), 512 itself with the plain loads of shorter rows.
  int ch = 1, wpr = 1;
  while (ch < 8 && ch * 512 < N) ch *= 2;
  while (ch * wpr * 512 < N) wpr *= 2;
  if (N == 16384) { ch = 16; wpr /= 2; }
  DeviceInfo di;
  if (!device_info(&di)) return;
  // A row that starts at any element, one of few: a wavefront's own work on it is the call's time, so it takes two vectors per
  // lane where the wavefronts are there for it.  LayerNorm, us: 16 x 2071 8.8 -> 4.6, 512 x 3001 9.0 -> 4.7, 16 x 5003 8.8 -> 4.5;
  // 2048 x 4097 and beyond are faster the other way.
  const int spread = ch * wpr / 2;
  const bool few = N % 8 != 0 && spread >= 2 && spread <= 8 && M * spread <= (int64_t)di.cus * 32;
  // Rows of exactly 4096 and 8192 always do, the next of a workgroup's rows in flight beside it; a lane with 8 or 16 vectors left a fraction
  // of the wavefronts.  us, before / so: RMSNorm 12288 x 4096 36.0 / 30.4, LayerNorm 12288 x 4096 39.7 / 31.3, 5120 x 8192 32.2 / 26.8,
  // 16384 x 8192 97 / 88; inference with K = 128, 8192 x 4096 54.9 / 47.6, 65536 x 8192 630 / 599.  (Between 1024 and 4096 rows of 4096 the
  // normalisation of GELU has too few rows for what a workgroup sets up: 2048 22.3 / 23.6.)  Other multiples of 8 keep a wavefront or two
  // per row.  So over that, 64 to 16384 rows: LayerNorm 2560 to 4088 columns 0.84 - 1.03 (mean 0.98), 5120 to 8184 0.93 - 1.03 (0.99),
  // RMSNorm 0.90 - 1.02 and 0.89 - 1.01, inference with K = 128 0.89 - 1.03 (0.95) and 0.91 - 1.12 (1.04).
  const bool whole = N == 8192 || (N == 4096 && (ACT != ACT_GELU || M <= 1024 || M >= 4096));
  if (few || whole) { ch = 2; wpr = spread; }
  const int fit = ch > 1 && N == (int64_t)ch * wpr * 512 ? FIT_FULL : (N % 8 == 0 ? FIT_VECTORS : FIT_ANY);
  // Where all workgroups walk the rows side by side, what they read and, rows behind, write keep one distance, and at some distances the
  // two get in each other's way.  From half as much again as the memory-side cache on, they walk stretches of the rows instead.
  // Stand-alone norms, one workgroup per compute unit, a stretch for each die: LayerNorm 65536 x 4096, us, at 13 distances between input and
  // output from 0 to 128 MB: a wavefront per row 189 - 193, two workgroups side by side 177 - 213, so 171 - 174 (one side by side 173 - 213, two so
  // 187 - 196); 65536 x 8192 382 - 391, 359 - 429, 349 - 365.  Side by side / so at a good distance: 16384 x 4096 45 / 48, 20000 54.8 / 55.0,
  // 24000 64.9 / 64.4, 10000 x 8192 55.6 / 55.3, 16384 88.5 / 86.4.
  // The block, two workgroups past the caches, three stretches (eight 186 - 198, one workgroup 210 - 219), unless it normalises in place: at
  // four distances, a wavefront per row / through the caches side by side / so: 24576 x 4096 78 - 82 77 - 78 73 - 74, 65536 x 4096 193 - 200 204 - 209
  // 187 - 191, 32768 x 8192 199 - 203 197 - 208 192 - 194, 65536 x 8192 399 - 404 407 - 424 378 - 392; 22000 x 4096 70 64 67, 11000 x 8192 77 67
  // 69; in place 65536 x 4096 196 167 197.
  const bool apart = whole && M * N * 4 >= kMemorySideCache / 2 * 3 && (ACT != ACT_GELU || Zsave != Y);
  // A stand-alone norm whose input and output together fill the memory-side cache runs past the caches.  4096 columns, us, through / past
  // them, buffers new to every pass: LayerNorm 8192 rows 25.0 / 24.8, 12288 38.6 / 35.1, 16384 49.0 / 45.5, 20480 61.9 / 56.4 (RMSNorm
  // 24.4 / 24.4, 38.1 / 34.7, 48.4 / 45.3, 61.3 / 56.4); the same buffers in every pass, which is how a layer finds what the one before it
  // wrote: 21.6 / 23.7, 31.3 / 34.7, 44.5 / 44.8, 61.5 / 55.9 (20.8 / 23.1, 30.3 / 33.6, 40.9 / 44.4, 60.6 / 55.7).  The line stands where the
  // two weigh the same.
  const bool past_caches = apart || (whole && ACT != ACT_GELU && M * N * 4 >= kMemorySideCache);
  const int nt = 512;
  // a workgroup of the widest variant fills a CU's register file; narrower rows leave room for more of them
  const int64_t per_wg = nt / 64 / wpr;
  int64_t wgs = (M + per_wg - 1) / per_wg;
  // (Stand-alone norms of 8192 columns: as many workgroups as gamma and beta leave room for in LDS.  With twice as many each sets those
  // up for half the rows, before the others end.  LayerNorm / RMSNorm, us, a wavefront per row / four / two per compute unit: 1536 rows
  // 10.6 11.7 10.5 / 9.5 10.1 9.0, 1792 11.3 12.6 11.3 / 10.2 11.5 10.3, 2304 18.5 15.8 13.7 / 15.9 13.6 12.5, 4096 21.8 22.8 22.0 / 21.3 20.9
  // 20.9, 6144 35.3 31.7 31.8 / 35.6 30.1 30.4.)
  const bool pair = past_caches || (N == 8192 && ACT != ACT_GELU);
  const int64_t per_cu = whole && !pair ? (ACT == ACT_GELU && N == 4096 ? 3 : 4)
                                              : (wpr == 8 || (ch == 2 && wpr > 1) ? 2 : (ch == 1 ? 8 : (16 / ch > wpr ? 16 / ch / wpr : 1)));
  const int64_t cap = (int64_t)di.cus * (apart && ACT != ACT_GELU ? 1 : per_cu);
  if (wgs > cap) wgs = cap;
  const int stretches = apart ? (ACT == ACT_GELU ? 3 : di.xcds) : 1;
  wgs -= wgs % stretches;            // (of many)
#define FDL_F2R(CHH, FIT, WPR)                                                                                        \
  launch_f2_rows_one<CHH, FIT, 512, ACT, WPR>(wgs, stretches, s, M, N, eps, (const bf16_t*)Zsave, gamma, beta, (bf16_t*)Y, mean, rstd)
#define FDL_F2R_FIT(FIT)                                                                                              \
  do {                                                                                                                \
    if (ch == 1) FDL_F2R(1, FIT, 1); else if (ch == 2) FDL_F2R(2, FIT, 1); else if (ch == 4) FDL_F2R(4, FIT, 1);        \
    else if (wpr == 1) FDL_F2R(8, FIT, 1);                                                                             \
    else if (wpr == 2) FDL_F2R(8, FIT, 2); else if (wpr == 4) FDL_F2R(8, FIT, 4); else FDL_F2R(8, FIT, 8);            \
  } while (0)
  if (few) {
    if (wpr == 2) FDL_F2R(2, FIT_ANY, 2); else if (wpr == 4) FDL_F2R(2, FIT_ANY, 4); else FDL_F2R(2, FIT_ANY, 8);
  } else if (past_caches) {
    if (wpr == 4) FDL_F2R(2, FIT_FULL, 4); else FDL_F2R(2, FIT_FULL, 8);
  } else if (whole) {
    if (wpr == 4) FDL_F2R(2, FIT_VECTORS, 4); else FDL_F2R(2, FIT_VECTORS, 8);
  } else if (fit == FIT_FULL) {
    // (1024, 2048, 16384 and 32768 columns; 4096 where `whole` leaves it)
    if (ch == 2) FDL_F2R(2, FIT_FULL, 1);
    else if (ch == 4) FDL_F2R(4, FIT_FULL, 1);
    else if (ch == 16) FDL_F2R(16, FIT_FULL, 2);
    else if (wpr == 8) FDL_F2R(8, FIT_FULL, 8);
    else if constexpr (ACT == ACT_GELU) FDL_F2R(8, FIT_FULL, 1);
  } else if (fit == FIT_VECTORS) {
    FDL_F2R_FIT(FIT_VECTORS);
  } else {
    FDL_F2R_FIT(FIT_ANY);
  }
#undef FDL_F2R_FIT
#undef FDL_F2R
}

// Which kernel normalises rows of N elements: bf16 rows up to 32768 go one to a wavefront or to two, four or eight of them,
// fp32 rows up to 16384 one to a workgroup that is as small as the row allows.  Longer ones are streamed by the stand-alone
// norms and dealt out in segments by the block (part: f2_part_bytes).
constexpr int64_t kRowsLimitBf16 = 32768, kRowsLimitF32 = 16384;
size_t f2_part_bytes(int dt, int64_t M, int64_t N) {
  if (N <= (dt == kF32 ? kRowsLimitF32 : kRowsLimitBf16)) return 0;
  const int64_t seg = dt == kF32 ? long_segment<float>() : long_segment<bf16_t>();
  return (size_t)M * (size_t)((N + seg - 1) / seg) * sizeof(double2);
}
template <class T, int ACT>
void launch_row_norm(int64_t M, int64_t N, float eps, const void* A, const float* gamma, const float* beta, void* Y,
                     float* mean, float* rstd, void* part, hipStream_t s) {
  constexpr int V = 16 / (int)sizeof(T);
  if constexpr (ACT == ACT_GELU) {
    if (N <= (sizeof(T) == 4 ? 64 : 128)) {
      const int64_t wgs = (M + 15) / 16;
      const dim3 grid((unsigned)(wgs < 2048 ? wgs : 2048));
#define FDL_NARROW(K) hipLaunchKernelGGL((f2_narrow_kernel<T, K>), grid, dim3(256), 0, s, M, N, eps, (const T*)A, gamma, beta, (T*)Y, mean, rstd)
      if (N <= 16) FDL_NARROW(1); else if (N <= 32) FDL_NARROW(2); else if (N <= 64) FDL_NARROW(4); else FDL_NARROW(8);
#undef FDL_NARROW
      return;
    }
  }
  if constexpr (sizeof(T) == 4) {
    const int64_t vectors = (N + V - 1) / V;
    // (GELU with up to two vectors a thread: 94 registers, most of them constants, five workgroups of 256 on a compute unit; with eight
    // of them in the grid forward passes of 80 shapes with 257 - 1024 columns were 2 - 4 % slower, 3630 x 64 x 913 31.1 to 30.3 us)
#define FDL_ROW(NT, S)                                                                                              \
  do {                                                                                                              \
    /* a full part's wavefronts, or what fits beside one another; any number is correct */                          \
    const int64_t cap = (int64_t)256 * (NT == 256 && S <= 2 && ACT == ACT_GELU ? 5 : 2048 / NT);                     \
    hipLaunchKernelGGL((row_wg_kernel<NT, S, ACT>), dim3((unsigned)(M < cap ? M : cap)), dim3(NT), 0, s, M, N, eps, \
                       (const T*)A, gamma, beta, (T*)Y, mean, rstd, F64Sums{});                                     \
    return;                                                                                                         \
  } while (0)
    // (stand-alone norms: three small trips through the caches beat workgroups that do not all fit, where there are more rows
    // than compute units and few for each.  LayerNorm, us, this way / in registers: 824 x 4424 9.0 / 14.5, 363 x 8424 9.2 / 11.7,
    // 2048 x 2680 11.1 / 12.7; 824 x 2048 6.3 / 4.9, 824 x 12000 23.9 / 22.4, 4096 x 4424 38.4 / 36.7, 128 x 5120 5.4 / 4.5)
    const bool streamed = ACT != ACT_GELU && N > 2048 && N <= 10240 && M > 256 && M <= 2048;
    if (!streamed) {
      if (vectors <= 64) FDL_ROW(64, 1);
      if (vectors <= 256) FDL_ROW(256, 1);
      if (vectors <= 512) FDL_ROW(256, 2);
      if (vectors <= 1024) FDL_ROW(256, 4);
      if (vectors <= 2048) FDL_ROW(512, 4);
      if (N <= kRowsLimitF32) FDL_ROW(1024, 4);
    }
#undef FDL_ROW
  } else if (N <= kRowsLimitBf16) {
    launch_rows_act<ACT>(M, N, eps, A, gamma, beta, Y, mean, rstd, s);
    return;
  }
  if constexpr (ACT == ACT_GELU) {
    const int64_t segments = (N + long_segment<T>() - 1) / long_segment<T>();
    int64_t rows = M * segments / 2048;
    if (rows < 1) rows = 1;
    const dim3 grid((unsigned)(segments * ((M + rows - 1) / rows)));
    double2* moments = static_cast<double2*>(part);
    auto first = N % V == 0 ? long_moments_kernel<T, false> : long_moments_kernel<T, true>;
    auto second = N % V == 0 ? long_apply_kernel<T, false> : long_apply_kernel<T, true>;
    hipLaunchKernelGGL(first, grid, dim3(256), 0, s, M, N, (int)segments, (int)rows, (const T*)A, moments);
    hipLaunchKernelGGL(second, grid, dim3(256), 0, s, M, N, (int)segments, (int)rows, eps, (const T*)A, moments, gamma, beta,
                       (T*)Y, mean, rstd);
    return;
  }
  const bool vec = N % V == 0 && ((uintptr_t)A | (uintptr_t)Y) % 16 == 0;
  const unsigned blocks = (unsigned)(M < 8192 ? M : 8192);
  if (vec) hipLaunchKernelGGL((row_stream_kernel<T, V, ACT>), dim3(blocks), dim3(256), 0, s, M, N, eps, (const T*)A, gamma, beta, (T*)Y, mean, rstd);
  else hipLaunchKernelGGL((row_stream_kernel<T, 1, ACT>), dim3(blocks), dim3(256), 0, s, M, N, eps, (const T*)A, gamma, beta, (T*)Y, mean, rstd);
}

// fp32 storage, rows of 65 to 2048 columns: the same from the parts of Z's tiles
bool f2_takes_sums(int64_t N) { return N > 64 && N <= 2048; }
void launch_f2_sums(int64_t M, int64_t N, float eps, const F64Sums& q, const float* gamma, const float* beta, void* Y, float* mean,
                    float* rstd, hipStream_t s) {
#define FDL_SUMS(NT, S)                                                                                                       \
  do {                                                                                                                        \
    const int64_t cap = (int64_t)256 * (2048 / NT);                                                                           \
    hipLaunchKernelGGL((row_wg_kernel<NT, S, ACT_GELU, true>), dim3((unsigned)(M < cap ? M : cap)), dim3(NT), 0, s, M, N,     \
                       eps, (const float*)q.Z, gamma, beta, (float*)Y, mean, rstd, q);                                        \
    return;                                                                                                                   \
  } while (0)
  if (N <= 256) FDL_SUMS(64, 1);
  if (N <= 1024) FDL_SUMS(256, 1);
  FDL_SUMS(256, 2);
#undef FDL_SUMS
}
void launch_f2(int dt, int64_t M, int64_t N, float eps, const void* Zsave, const float* gamma, const float* beta, void* Y,
               float* mean, float* rstd, void* part, hipStream_t s) {
  if (dt == kF32) launch_row_norm<float, ACT_GELU>(M, N, eps, Zsave, gamma, beta, Y, mean, rstd, part, s);
  else launch_row_norm<bf16_t, ACT_GELU>(M, N, eps, Zsave, gamma, beta, Y, mean, rstd, part, s);
}

// Y = LayerNorm(A) gamma + beta over the last dimension; mean, rstd [M] out
void launch_layernorm(int dt, int64_t M, int64_t N, float eps, const void* A, const float* gamma, const float* beta,
                      void* Y, float* mean, float* rstd, hipStream_t s) {
  if (dt == kF32) launch_row_norm<float, ACT_NONE>(M, N, eps, A, gamma, beta, Y, mean, rstd, nullptr, s);
  else launch_row_norm<bf16_t, ACT_NONE>(M, N, eps, A, gamma, beta, Y, mean, rstd, nullptr, s);
}

// Y = A (mean(A^2) + eps)^-1/2 weight over the last dimension
void launch_rmsnorm(int dt, int64_t M, int64_t N, float eps, const void* A, const float* weight, void* Y, hipStream_t s) {
  if (dt == kF32) launch_row_norm<float, ACT_RMS>(M, N, eps, A, weight, weight, Y, nullptr, nullptr, nullptr, s);
  else launch_row_norm<bf16_t, ACT_RMS>(M, N, eps, A, weight, weight, Y, nullptr, nullptr, nullptr, s);
}

// groups of the first stage of a column sum over M rows
int colsum_groups(int64_t M) { return (int)(M < 256 ? (M > 0 ? M : 1) : 256); }

// sums over the rows of G [M][N], pitch ldg: colsum_groups(M) partial sums per column, then the sums themselves
void launch_colsum_partial(int dt, int64_t M, int64_t N, int64_t ldg, const void* G, bool blocked, void* colpart, hipStream_t s) {
  const int groups = colsum_groups(M);
  const int vmax = dt == kF32 ? 4 : 8;
  const bool vec = ldg % vmax == 0;            // (a vector that passes N stays inside the pitch)
  const int V = vec ? vmax : 1;
  const int strips = (int)((N + 256 * (int64_t)V - 1) / (256 * (int64_t)V));
  const dim3 grid((unsigned)(strips * groups));
  if (dt == kF32) {
    auto kern = vec ? colsum_partial_kernel<float, 4> : colsum_partial_kernel<float, 1>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, M, N, ldg, strips, groups, (const float*)G, (double*)colpart);
  } else {
    auto kern = vec && blocked ? colsum_partial_kernel<bf16_t, 8, true> : (vec ? colsum_partial_kernel<bf16_t, 8> : colsum_partial_kernel<bf16_t, 1>);
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, M, N, ldg, strips, groups, (const bf16_t*)G, (float*)colpart);
  }
}
void launch_colsum_finish(int64_t M, int64_t N, const void* colpart, float* out, hipStream_t s) {
  hipLaunchKernelGGL(b2_kernel, dim3((unsigned)((N + 63) / 64), 1), dim3(1024), 0, s, N, colsum_groups(M), (const float*)colpart,
                     out, out, out);
}

// H = SiLU(G) * U over n elements (H may alias G or U)
void launch_silu_mul(int dt, int64_t n, const void* G, const void* U, void* H, hipStream_t s) {
  const int vmax = dt == kF32 ? 4 : 8;
  const bool vec = n % vmax == 0 && ((uintptr_t)G | (uintptr_t)U | (uintptr_t)H) % 16 == 0;
  const int64_t per = 256 * (int64_t)(vec ? vmax : 1);
  int64_t blocks = (n + per - 1) / per;
  if (blocks > 16384) blocks = 16384;
  if (blocks < 1) blocks = 1;
  if (dt == kF32) {
    if (vec) hipLaunchKernelGGL((silu_mul_kernel<float, 4>), dim3((unsigned)blocks), dim3(256), 0, s, n, (const float*)G, (const float*)U, (float*)H);
    else hipLaunchKernelGGL((silu_mul_kernel<float, 1>), dim3((unsigned)blocks), dim3(256), 0, s, n, (const float*)G, (const float*)U, (float*)H);
  } else {
    if (vec) hipLaunchKernelGGL((silu_mul_kernel<bf16_t, 8>), dim3((unsigned)blocks), dim3(256), 0, s, n, (const bf16_t*)G, (const bf16_t*)U, (bf16_t*)H);
    else hipLaunchKernelGGL((silu_mul_kernel<bf16_t, 1>), dim3((unsigned)blocks), dim3(256), 0, s, n, (const bf16_t*)G, (const bf16_t*)U, (bf16_t*)H);
  }
}

void launch_b1a(int dt, int64_t M, int64_t N, const void* dY, const void* Zsave, const float* gamma, const float* mean,
                const float* rstd, void* c12, hipStream_t s) {
  if (dt == kF32) b1a_impl<float>(M, N, dY, Zsave, gamma, mean, rstd, c12, s);
  else b1a_impl<bf16_t>(M, N, dY, Zsave, gamma, mean, rstd, c12, s);
}

void launch_b1b(int dt, int64_t M, int64_t N, int64_t ldz, int rows_per_group, int groups, const void* dY, const void* Zsave,
                const float* gamma, const float* mean, const float* rstd, const void* c12, void* dZ, void* colpart,
                hipStream_t s) {
  if (dt == kF32) b1b_impl<float>(M, N, ldz, rows_per_group, groups, dY, Zsave, gamma, mean, rstd, c12, dZ, colpart, s);
  else b1b_impl<bf16_t>(M, N, ldz, rows_per_group, groups, dY, Zsave, gamma, mean, rstd, c12, dZ, colpart, s);
}

// dZ [M][ldz]: zero the surplus columns [N, ldz) of every row (padded mode of the fast contractions)
namespace {
__global__ __launch_bounds__(256) void zero_cols_kernel(unsigned short* __restrict__ dZ, int64_t M, int64_t N, int64_t ldz) {
  const int64_t w = ldz - N, n = M * w;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / w, c = i - r * w;
    dZ[r * ldz + N + c] = 0;
  }
}
}  // namespace
void launch_zero_cols_bf16(void* dZ, int64_t M, int64_t N, int64_t ldz, hipStream_t s) {
  if (ldz <= N || M <= 0) return;
  int64_t blocks = (M * (ldz - N) + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(zero_cols_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (unsigned short*)dZ, M, N, ldz);
}

bool b1_fused_supported(int dt, int64_t N, int64_t ldz) { return fused_threads(dt, N, ldz) != 0; }

int b1_fused_slots(int dt, int64_t N, int64_t ldz) { return b1_slots(dt, N, ldz); }

// Row groups (= workgroups) of the fused kernel.  Each group leaves 3 N partial column sums behind and pays for its start
// (the table, the first rows), so fewer groups mean less traffic for the phase and for the column reduction after it;
// more of them hide the chain of each row's reductions behind one another.  Measured with the column reduction, us, for
// 256 / 512 / 1024 groups: bf16 3001 x 1537: 26.2 / 23.3 / 28.1; 32768 x 1024: 103 / 72.8 / 65.4; 16384 x 4096: 85.3 / 82.0
// / 88.9; 65536 x 8192: 578 / 569 / 578; 1000 x 5000: 22.3 / 28.5.  fp32 rows of more than 1024 columns, whose fp64 arithmetic
// fills the vector units with one workgroup of 512 threads (four columns each, eight above 2048) per compute unit: whole
// backward passes with K = 8, 256 / 512 groups, 3001 x 1537 62.3 / 66.4, 8192 x 4096 243 / 255, 500 x 2292 40.2 / 46.6; 256 are
// faster on all of 65 shapes, by 1 % (30000 rows) to 17 % (a thousand and fewer).
int b1_fused_groups(int dt, int64_t M, int64_t N) {
  const int nt = fused_threads(dt, N, N);
  if (dt == kF32 && nt > 256) return 256;
  if (nt <= 256 && M >= 16 * 1024) return 1024;
  return M >= (nt < 1024 ? 5 : 16) * 512 ? 512 : 256;
}

// Rows per group of the two-kernel path: about 1024 workgroups, but at least 16 rows each (partial column sums as above;
// bf16 4096 x 16384 with the column reduction: 16 rows 157 us, 32 146, 64 155; 1273 x 14080: 8 rows 44.9, 16 42.0, 32 48.2).
// For bf16 a group's sums are fp32 chains of that many rows, which meet in fp64: 65536 x 16384 has chains of 512, and dgamma, db
// and dbeta are 4.3e-8, 4.0e-8 and 2.7e-8 from 64 bits there (relative 2-norm; rounding the result alone is 2.7e-8; chains of 64
// with a polynomial for the CDF were at 5.4e-7, 9.1e-8 and 2.7e-8).  Chains of 16 folded into fp64 reach 2.8e-8, 2.7e-8 and 2.7e-8
// and cost the whole step 1 - 2 %.
int b1b_rows_per_group(int dt, int64_t M, int64_t N) {
  const int64_t width = 256 * (dt == kF32 ? 4 : 8), strips = (N + width - 1) / width;
  int64_t rpg = M * strips / 1024;
  if (rpg < 16) rpg = 16;
  if (rpg < (M + 1023) / 1024) rpg = (M + 1023) / 1024;     // at most 1024 groups' worth of partial sums
  return (int)rpg;
}

void launch_b1_fused(int dt, int64_t M, int64_t N, int64_t ldz, int groups, bool blocked, const void* dY, const void* Zsave,
                     const float* gamma, const float* mean, const float* rstd, void* dZ, void* colpart, hipStream_t s) {
  if (dt == kF32) b1_fused_impl<float>(M, N, ldz, groups, false, dY, Zsave, gamma, mean, rstd, dZ, colpart, s);
  else b1_fused_impl<bf16_t>(M, N, ldz, groups, blocked, dY, Zsave, gamma, mean, rstd, dZ, colpart, s);
}

void launch_b2(int64_t N, int groups, const void* colpart, float* dbeta, float* dgamma, float* db, hipStream_t s) {
  hipLaunchKernelGGL(b2_kernel, dim3((unsigned)((N + 63) / 64), 3), dim3(1024), 0, s, N, groups, (const float*)colpart, dbeta,
                     dgamma, db);
}

void launch_finish(TailSums j, hipStream_t s) {
  unsigned blocks = 0;
  for (int k = 0; k < 2; k++) {
    j.blocks[k] = j.parts[k] > 0 ? (int)(((j.n[k] + 3) / 4 + 1023) / 1024) : 0;
    j.stride[k] = partial_stride(j.n[k]);
    blocks += (unsigned)j.blocks[k];
  }
  blocks += (unsigned)j.kinds * (unsigned)((j.N + 63) / 64);
  hipLaunchKernelGGL(finish_kernel, dim3(blocks), dim3(1024), 0, s, j);
}

}  // namespace fdl
