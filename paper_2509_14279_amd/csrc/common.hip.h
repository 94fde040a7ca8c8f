// Shared device-side helpers for the fused dense-layer kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fdl {

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int kWave = 64;

// Storage type -> arithmetic type: one level above the storage precision.
template <class T> struct ComputeOf;
template <> struct ComputeOf<float> { typedef double type; };
template <> struct ComputeOf<bf16_t> { typedef float type; };

template <class T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return (float)v; }

// Round a value of the arithmetic type to the storage type (nearest, ties to even).
template <class T, class C> __device__ __forceinline__ T to_storage(C v);
template <> __device__ __forceinline__ float to_storage<float, double>(double v) { return (float)v; }
template <> __device__ __forceinline__ float to_storage<float, float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t to_storage<bf16_t, float>(float v) { return (bf16_t)v; }
template <> __device__ __forceinline__ bf16_t to_storage<bf16_t, double>(double v) { return (bf16_t)(float)v; }

// ---------------------------------------------------------------------------------------------
// The normal distribution's CDF Phi and density phi are the two pieces of GELU_erf and its derivative:
//   GELU(z) = z Phi(z),   GELU'(z) = Phi(z) + z phi(z).
// fp32 storage evaluates them in fp64 (NormalTable), bf16 storage reads them from the table below; every
// row kernel does it through ActTable, so that the forward statistics, the values normalised and the backward pass agree
// exactly (for a constant row, rstd = eps^-1/2 multiplies any difference between them into Ahat).

// ---------------------------------------------------------------------------------------------
// Compile-time evaluation of the normal distribution in double precision (for the table below: its entries are
// constants, so the compiler computes them once instead of every workgroup at every launch).
namespace ctmath {
constexpr double kLn2 = 0.69314718055994530941723212145818;
constexpr double kInvSqrtPi = 0.56418958354775628694807945156077;
// exp(-t), t >= 0: -t = -k ln 2 - r with |r| <= ln2 / 2, a 24-term series for exp(-r), then k halvings
constexpr double exp_neg(double t) {
  if (t > 700.0) return 0.0;
  const long k = (long)(t / kLn2 + 0.5);
  const double r = t - (double)k * kLn2;
  double term = 1.0, sum = 1.0;
  for (int n = 1; n <= 24; n++) { term *= -r / (double)n; sum += term; }
  for (long i = 0; i < k; i++) sum *= 0.5;
  return sum;
}
// erf(x), x >= 0: the Maclaurin series below 2.5 (its largest term is about e^6, so cancellation costs 3 of 16 digits),
// 1 - erfc(x) from the continued fraction erfc(x) = exp(-x^2) / sqrt(pi) / (x + (1/2)/(x + 1/(x + (3/2)/(x + ...)))) above
constexpr double erf_pos(double x) {
  if (x < 2.5) {
    const double x2 = x * x;
    double term = x, sum = x;
    for (int n = 1; n <= 90; n++) {
      term *= -x2 / (double)n;
      sum += term / (double)(2 * n + 1);
    }
    return 2.0 * kInvSqrtPi * sum;
  }
  double f = x;
  for (int n = 120; n >= 1; n--) f = x + 0.5 * (double)n / f;
  return 1.0 - exp_neg(x * x) * kInvSqrtPi / f;
}
}  // namespace ctmath

// ---------------------------------------------------------------------------------------------
// Exact Phi for bf16 arguments, from a table in LDS.  A bf16 number has 8 significant bits, so the magnitudes in
// [2^-14, 16) are only 18 binades x 128 = 2304 values; for each of them the table holds
//   H = Phi(|z|) - 1/2      and (kPair) Q = |z| phi(|z|),
// both odd in z, as fp32 roundings of an fp64 evaluation.  Smaller magnitudes use the first entry (H, Q < 2.5e-5)
// and larger ones the last (H = 1/2, Q = 0 to fp32).  A lookup is: clamp the magnitude bits, one LDS read, copy
// the sign of z onto the entries - five integer instructions, and GELU(z) = z (1/2 + sign(z) H) carries no approximation error beyond fp32 rounding.  The entries are compile-time
// constants in device memory; every workgroup copies them into its LDS (coalesced, a few KB from the L2).
constexpr uint32_t kGaussLo = 0x3880u;          // bf16 bits of 2^-14
constexpr uint32_t kGaussHi = 0x417fu;          // bf16 bits of the largest bf16 number below 16
constexpr int kGaussEntries = (int)(kGaussHi - kGaussLo) + 1;
struct GaussTableData { alignas(16) float h[kGaussEntries]; alignas(16) float pair[2 * kGaussEntries]; };
constexpr GaussTableData make_gauss_table() {
  GaussTableData t = {};
  for (int i = 0; i < kGaussEntries; i++) {
    const double z = (double)__builtin_bit_cast(float, (kGaussLo + (uint32_t)i) << 16);
    const double H = 0.5 * ctmath::erf_pos(z * 0.70710678118654752440);
    const double Q = z * ctmath::exp_neg(0.5 * z * z) * 0.39894228040143267794;
    t.h[i] = (float)H;
    t.pair[2 * i] = (float)H;
    t.pair[2 * i + 1] = (float)Q;
  }
  return t;
}
__device__ const GaussTableData g_gauss_table = make_gauss_table();

template <bool kPair> struct GaussTable {
  static constexpr uint32_t kLo = kGaussLo;
  static constexpr uint32_t kHi = kGaussHi;
  static constexpr int kEntries = kGaussEntries;
  static constexpr int kEntryBytes = kPair ? 8 : 4;
  static constexpr int kBytes = kEntries * kEntryBytes;

  // tbl: LDS; every thread of the workgroup calls this (followed by a barrier at the caller)
  static __device__ __forceinline__ void build(float* tbl, int tid, int nthreads) {
    const f32x4* src = reinterpret_cast<const f32x4*>(kPair ? g_gauss_table.pair : g_gauss_table.h);
    constexpr int kVectors = kBytes / 16;
    static_assert(kBytes % 16 == 0, "whole vectors");
#pragma unroll 8
    for (int i = tid; i < kVectors; i += nthreads) reinterpret_cast<f32x4*>(tbl)[i] = src[i];
  }
  // LDS address of the entry for the bf16 number whose bits (sign included or not) are in the low 16 bits of
  // `bits`: clamped magnitude bits times the entry size plus origin(table address), in three instructions
  static __device__ __forceinline__ uint32_t origin(uint32_t table_lds_address) {
    return table_lds_address - kLo * (uint32_t)kEntryBytes;     // wraps; the sum below is the true address again
  }
  static __device__ __forceinline__ uint32_t address_of(uint32_t bits, uint32_t org) {
    uint32_t mag = bits & 0x7fffu;
    mag = mag < kLo ? kLo : mag;
    mag = mag > kHi ? kHi : mag;
    return mag * (uint32_t)kEntryBytes + org;
  }
  // sign(z) |h|: magnitude bits of h, sign bit of z
  static __device__ __forceinline__ float with_sign_of(float h, float z) {
    return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, h) & 0x7fffffffu) |
                                         (__builtin_bit_cast(uint32_t, z) & 0x80000000u));
  }
};

// ---------------------------------------------------------------------------------------------
// Phi and phi in fp64 (fp32 storage), from a table in LDS and two short series.  Node k holds Phi(-c) and phi(c) at c = k / 64;
// a = |z| lies h = a - c, |h| <= 1/128, from the nearest one.  With m = c + h/2 the middle and 1 + e = phi(m) / phi(c):
//   e = exp(-h (c + h/4) / 2) - 1, eight terms;   phi(z) = phi(c) (1 + e)^2 exp(-h^2 / 4);
//   Phi(-a) = Phi(-c) - integral of phi from c to a
//           = Phi(-c) - phi(m) h (1 + (m^2 - 1) h^2 / 24 + (m^4 - 6 m^2 + 3) h^4 / 1920 + (m^6 - 15 m^4 + 45 m^2 - 15) h^6 / 322560),
// the Taylor expansion about the middle (phi's even derivatives are Hermite polynomials times phi).  Beyond the last node, at
// 13.25: exp, and the asymptotic series Phi(-a) = phi(a) / a (1 - 1/a^2 + 1 3 / a^4 - 1 3 5 / a^6 + ...), thirteen terms.
// Largest relative error, here / 0.5 erfc(-z / sqrt 2) and exp(-z^2 / 2) / sqrt(2 pi) of a library: Phi(-a), a to 1.5 2.2e-16 /
// 6e-16, to 4.5 2.0e-16 / 3e-15, to 9 2.7e-16 / 1.1e-14, to 13.25 8e-16 / 2.9e-14, beyond 4.4e-16 / 1.7e-13 (the argument's rounding);
// phi 2.1e-16 / 2.5e-16, beyond 2.8e-16 / 2.5e-16.
// The row kernels of fp32 storage are bound by this arithmetic: some 35 fp64 instructions (45 with phi) and one branch a vector,
// where the library's erfc and exp go through several ranges per wavefront.  3001 x 1537, us: normalisation 26 -> 18, backward row
// pass 42 -> 28 (with one polynomial of degree 20 for the whole axis and exp's, no table: 20 and 36).  Six terms and two, zero
// beyond the table: 4e-13 from Phi and phi at 13 and no gradient at all beyond, for whole fp32 steps 1 % faster and forward passes of
// short reductions 2 - 3 % (257 - 1024 columns, where 64 instead of 94 registers let eight workgroups share a compute unit, 2 - 8 %).
namespace ctmath {
// Sums and products of two doubles each (hi + lo), where the table's entries are to be correctly rounded
struct Two { double hi, lo; };
constexpr Two two_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
constexpr Two operator+(Two a, Two b) {
  const Two s = two_sum(a.hi, b.hi);
  return two_sum(s.hi, s.lo + (a.lo + b.lo));
}
constexpr double low_part(double a, double b, double p) {      // a b - p, p the rounded product: halves of 26 bits each (Dekker)
  const double s = 134217729.0, ta = s * a, ah = ta - (ta - a), al = a - ah, tb = s * b, bh = tb - (tb - b), bl = b - bh;
  return ((ah * bh - p) + ah * bl + al * bh) + al * bl;
}
constexpr Two operator*(Two a, Two b) {
  const double p = a.hi * b.hi;
  return two_sum(p, low_part(a.hi, b.hi, p) + (a.hi * b.lo + a.lo * b.hi));
}
// phi(c) = exp(-c^2 / 2) / sqrt(2 pi), c a multiple of 2^-7 below 2^4 (its square is exact): c^2 / 2 = k ln 2 + r, ln 2 in 24 bits
// and the rest, so that r is exact to 10^-22; 24 terms, then k halvings
constexpr Two normal_density(double c) {
  const double t = 0.5 * c * c;
  const long k = (long)(t / 0.69314718055994531 + 0.5);
  const Two r = two_sum((double)k * 0.693147182464599609375 - t, (double)k * -1.904654299957767878542e-9);   // -r
  Two sum = {1.0, 0.0};
  for (int n = 24; n >= 1; n--) {
    const Two x = r * sum;
    const double q = x.hi / (double)n, p = q * (double)n;
    sum = Two{1.0, 0.0} + two_sum(q, ((x.hi - p) - low_part(q, (double)n, p) + x.lo) / (double)n);
  }
  sum = sum * Two{0x1.9884533d43651p-2, -0x1.cbc0d30ebfd15p-56};
  for (long i = 0; i < k; i++) { sum.hi *= 0.5; sum.lo *= 0.5; }
  return sum;
}
}  // namespace ctmath
constexpr int kNormalNodes = 848;               // up to 13.25
struct NormalNode { double tail, density; };
struct NormalTableData { alignas(16) NormalNode node[kNormalNodes + 1]; };
constexpr NormalTableData make_normal_table() {
  NormalTableData t = {};
  // Phi(-13.25) from the continued fraction phi(x) / (x + 1 / (x + 2 / (x + ...))), then the integral from node to node, downwards
  const double top = (double)kNormalNodes / 64.0;
  double f = top;
  for (int n = 60; n >= 1; n--) f = top + (double)n / f;
  const ctmath::Two d = ctmath::normal_density(top);
  ctmath::Two sum = {d.hi / f, 0.0};
  t.node[kNormalNodes] = {sum.hi, d.hi};
  for (int k = kNormalNodes - 1; k >= 0; k--) {
    const double c = (double)k / 64.0, h = 1.0 / 64.0, m = c + 0.5 * h, m2 = m * m, h2 = h * h;
    const double rest = h2 * ((m2 - 1.0) / 24.0 +
                              h2 * ((m2 * (m2 - 6.0) + 3.0) / 1920.0 +
                                    h2 * ((((m2 - 15.0) * m2 + 45.0) * m2 - 15.0) / 322560.0 +
                                          h2 * ((((m2 - 28.0) * m2 + 210.0) * m2 - 420.0) * m2 + 105.0) / 92897280.0)));
    sum = sum + ctmath::normal_density(m) * ctmath::two_sum(h, h * rest);
    t.node[k] = {sum.hi, ctmath::normal_density(c).hi};
  }
  return t;
}
__device__ const NormalTableData g_normal_table = make_normal_table();

// Phi(-a) and (DENSITY) phi(a), a - h a node with the two values given
template <bool DENSITY>
__device__ __forceinline__ void normal_near(double a, double h, double tail, double density, double& q, double& phi) {
  const double m = __builtin_fma(h, -0.5, a), mh = m * h, h2 = h * h, w = mh * mh, v = __builtin_fma(h2, -0.25, mh);
  double e = 1.0 / 10321920.0;
  e = __builtin_fma(e, v, -1.0 / 645120.0);
  e = __builtin_fma(e, v, 1.0 / 46080.0);
  e = __builtin_fma(e, v, -1.0 / 3840.0);
  e = __builtin_fma(e, v, 1.0 / 384.0);
  e = __builtin_fma(e, v, -1.0 / 48.0);
  e = __builtin_fma(e, v, 0.125);
  e = __builtin_fma(e, v, -0.5) * v;
  double s = __builtin_fma(w, 1.0 / 322560.0, __builtin_fma(h2, -15.0 / 322560.0, 1.0 / 1920.0));
  s = __builtin_fma(w, s, __builtin_fma(h2, -6.0 / 1920.0, 1.0 / 24.0));
  s = __builtin_fma(w, s, h2 * __builtin_fma(h2, 3.0 / 1920.0, -1.0 / 24.0));
  const double step = __builtin_fma(density, e, density) * h;
  q = tail - __builtin_fma(step, s, step);
  if (DENSITY) {
    const double g = h2 * __builtin_fma(h2, __builtin_fma(h2, -1.0 / 384.0, 1.0 / 32.0), -0.25), p = __builtin_fma(e, e, e + e);
    phi = __builtin_fma(density, __builtin_fma(g, p, g + p), density);
  }
}
// and beyond the last node.  Seldom taken: rolled loops, and a count the compiler cannot move out of the caller's loops, keep this
// from costing the usual path registers.  exp(-t), t = a^2 / 2 (exact): t = k ln 2 + r, the Taylor series of exp(-r), k halvings.
// From 39 on both are zero: larger arguments, infinity among them, count as 52 (beyond 10^8 nothing would be left of r).
template <bool DENSITY> __device__ __forceinline__ void normal_tail(double a, double& q, double& phi) {
  int terms = 13;
  asm volatile("" : "+s"(terms));
  a = __builtin_fmin(a, 52.0);
  const double t = 0.5 * (a * a), k = __builtin_rint(t * 1.44269504088896340736);
  const double r = __builtin_fma(k, 1.9046542999577680453e-9, __builtin_fma(k, -0.693147182464599609375, t));
  const double x = 1.0 / a, u = x * x;
  double d = 1.0, s = 1.0;
#pragma unroll 1
  for (int n = terms; n >= 1; n--) {
    d = __builtin_fma(d, -r / (double)n, 1.0);
    s = __builtin_fma(s, (1.0 - 2.0 * (double)n) * u, 1.0);
  }
  d = __builtin_ldexp(d * 0.39894228040143267794, -(int)k);
  q = d * x * s;
  if (DENSITY) phi = d;
}

struct NormalTable {
  static constexpr double kLast = (double)kNormalNodes / 64.0;
  typedef __attribute__((address_space(3))) const double lds_double;
  uint32_t base;
  template <int NT> __device__ __forceinline__ void build() {
    __shared__ __attribute__((aligned(16))) double tbl[2 * (kNormalNodes + 1)];
    const f32x4* src = reinterpret_cast<const f32x4*>(g_normal_table.node);
#pragma unroll 4
    for (int i = threadIdx.x; i <= kNormalNodes; i += NT) reinterpret_cast<f32x4*>(tbl)[i] = src[i];
    base = (uint32_t)(uintptr_t)(lds_double*)tbl;
    __syncthreads();
  }
  // up to the last node
  template <bool DENSITY> __device__ __forceinline__ void eval(double z, double& Phi, double& phi) const {
    const double a = __builtin_fmin(__builtin_fabs(z), kLast);
    // (the sum's last bits are the nearest node's number)
    const double magic = 0x1.8p52, t = __builtin_fma(a, 64.0, magic), k = t - magic;
    const uint32_t at = base + ((uint32_t)__builtin_bit_cast(uint64_t, t) << 4);
    typedef __attribute__((ext_vector_type(2))) double f64x2;
    const f64x2 node = *(const __attribute__((address_space(3))) f64x2*)(uintptr_t)at;
    double q;
    normal_near<DENSITY>(a, __builtin_fma(k, -1.0 / 64.0, a), node[0], node[1], q, phi);
    Phi = z > 0.0 ? 1.0 - q : q;               // (NaN: q is a small number; z Phi and z phi are NaN)
  }
  // whether z lies beyond it, and the values there
  template <bool DENSITY> static __device__ __forceinline__ bool far(double z, double& Phi, double& phi) {
    const bool is = __builtin_fabs(z) > kLast;
    if (__builtin_expect(is, 0)) {
      double q;
      normal_tail<DENSITY>(__builtin_fabs(z), q, phi);
      Phi = z > 0.0 ? 1.0 - q : q;
    }
    return is;
  }
};

// What the row kernels ask; both tables live in the workgroup's LDS (kPair: with z phi(z), for the backward pass).  NT: threads of the workgroup.
template <class T, bool kPair, int NT> struct ActTable;
template <bool kPair, int NT> struct ActTable<float, kPair, NT> {
  NormalTable tab;
  // every thread of the workgroup calls this; ends with a barrier
  __device__ __forceinline__ void build() { tab.build<NT>(); }
  // One branch for a thread's vector: seldom taken as it is, a branch per element keeps the elements' chains from overlapping
  // (forward passes up to 12 % slower).
  template <int V, class R> __device__ __forceinline__ void gelu(R z, double (&a)[V]) const {
    double phi;
#pragma unroll
    for (int v = 0; v < V; v++) {
      double Phi;
      tab.eval<false>((double)z[v], Phi, phi);
      a[v] = (double)z[v] * Phi;
    }
    if (__builtin_expect(some_far<V>(z), 0)) {
#pragma unroll
      for (int v = 0; v < V; v++) {
        double Phi = 0.0;
        if (NormalTable::far<false>((double)z[v], Phi, phi)) a[v] = (double)z[v] * Phi;
      }
    }
  }
  template <int V, class R> __device__ __forceinline__ void eval(R z, double (&Phi)[V], double (&zphi)[V]) const {
#pragma unroll
    for (int v = 0; v < V; v++) eval((double)z[v], false, Phi[v], zphi[v]);
    if (__builtin_expect(some_far<V>(z), 0)) {
#pragma unroll
      for (int v = 0; v < V; v++) {
        double phi;
        if (NormalTable::far<true>((double)z[v], Phi[v], phi)) zphi[v] = (double)z[v] * phi;
      }
    }
  }
  // Element by element, where registers are short.  far: what some_far says of the vector that z is of (uniform over the
  // wavefront: a scalar branch)
  template <int V, class R> static __device__ __forceinline__ bool some_far(R z) {
    float most = 0.0f;
#pragma unroll
    for (int v = 0; v < V; v++) most = __builtin_fmaxf(most, __builtin_fabsf(z[v]));
    return __builtin_amdgcn_ballot_w64(most > (float)NormalTable::kLast) != 0;
  }
  // far: what some_far says of the vector that z is of
  __device__ __forceinline__ void eval(double z, bool far, double& Phi, double& zphi) const {
    double phi;
    tab.eval<true>(z, Phi, phi);
    if (__builtin_expect(far, 0)) (void)NormalTable::far<true>(z, Phi, phi);
    zphi = z * phi;
  }
};
template <bool kPair, int NT> struct ActTable<bf16_t, kPair, NT> {
  typedef GaussTable<kPair> GT;
  typedef __attribute__((address_space(3))) float lds_float;
  typedef __attribute__((address_space(3))) f32x2 lds_f32x2;
  uint32_t org;
  // every thread of the workgroup calls this; ends with a barrier
  __device__ __forceinline__ void build() {
    __shared__ __attribute__((aligned(16))) float tbl[(kPair ? 2 : 1) * GT::kEntries];
    GT::build(tbl, threadIdx.x, NT);
    org = GT::origin((uint32_t)(uintptr_t)(const lds_float*)tbl);
    __syncthreads();
  }
  // z: a bf16 number
  __device__ __forceinline__ float gelu(float z) const {
    const float h = *(const lds_float*)(uintptr_t)GT::address_of(__builtin_bit_cast(uint32_t, z) >> 16, org);
    return z * (0.5f + GT::with_sign_of(h, z));
  }
  template <int V, class R> __device__ __forceinline__ void gelu(R z, float (&a)[V]) const {
#pragma unroll
    for (int v = 0; v < V; v++) a[v] = gelu(to_f32<bf16_t>(z[v]));
  }
  template <int V, class R> static __device__ __forceinline__ bool some_far(R) { return false; }
  template <int V, class R> __device__ __forceinline__ void eval(R z, float (&Phi)[V], float (&zphi)[V]) const {
#pragma unroll
    for (int v = 0; v < V; v++) eval(to_f32<bf16_t>(z[v]), false, Phi[v], zphi[v]);
  }
  __device__ __forceinline__ void eval(float z, bool, float& Phi, float& zphi) const {
    const f32x2 e = *(const lds_f32x2*)(uintptr_t)GT::address_of(__builtin_bit_cast(uint32_t, z) >> 16, org);
    Phi = 0.5f + GT::with_sign_of(e[0], z);
    zphi = GT::with_sign_of(e[1], z);
  }
};

// ---------------------------------------------------------------------------------------------
// Sums over the wavefronts that share a row pass through LDS: each wavefront writes its part into a slot, meets one barrier
// and reads the others' parts.  With one barrier per sum two consecutive sums must not share a slot: a wavefront may write the
// next sum's slot while another still reads this one's, and only the barrier after that shows that it is done.  So the two
// slots take turns from sum to sum, across rows: sum k of trip t of a walk with so many sums per row.
constexpr int row_sum_slot(int sums_per_row, int trip, int k) { return (sums_per_row * trip + k) & 1; }

// ---------------------------------------------------------------------------------------------
// Vector access helpers: V consecutive storage elements <-> V values of the arithmetic type.
template <class T, int V> struct VecIO;

template <> struct VecIO<float, 4> {
  template <class C> static __device__ __forceinline__ void load(const float* p, C (&v)[4]) {
    const f32x4 t = *reinterpret_cast<const f32x4*>(p);
    v[0] = (C)t[0]; v[1] = (C)t[1]; v[2] = (C)t[2]; v[3] = (C)t[3];
  }
  template <class C> static __device__ __forceinline__ void store(float* p, const C (&v)[4]) {
    f32x4 t; t[0] = (float)v[0]; t[1] = (float)v[1]; t[2] = (float)v[2]; t[3] = (float)v[3];
    *reinterpret_cast<f32x4*>(p) = t;
  }
};
template <> struct VecIO<float, 1> {
  template <class C> static __device__ __forceinline__ void load(const float* p, C (&v)[1]) { v[0] = (C)p[0]; }
  template <class C> static __device__ __forceinline__ void store(float* p, const C (&v)[1]) { p[0] = (float)v[0]; }
};
template <> struct VecIO<bf16_t, 8> {
  template <class C> static __device__ __forceinline__ void load(const bf16_t* p, C (&v)[8]) {
    const bf16x8 t = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = (C)(float)t[i];
  }
  template <class C> static __device__ __forceinline__ void store(bf16_t* p, const C (&v)[8]) {
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 8; i++) t[i] = (bf16_t)(float)v[i];
    *reinterpret_cast<bf16x8*>(p) = t;
  }
};
template <> struct VecIO<bf16_t, 1> {
  template <class C> static __device__ __forceinline__ void load(const bf16_t* p, C (&v)[1]) { v[0] = (C)(float)p[0]; }
  template <class C> static __device__ __forceinline__ void store(bf16_t* p, const C (&v)[1]) { p[0] = (bf16_t)(float)v[0]; }
};

// Sum over the 64 lanes of a wavefront; every lane receives the total.
template <class C> __device__ __forceinline__ C wave_sum(C v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
  return v;
}

// fp32: data-parallel-primitive lane moves folded into the adds instead of LDS permutes.
// dpp_f<CTRL, ROW_MASK>(x): the value of the lane CTRL selects; lanes in rows outside ROW_MASK read 0.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROW_MASK, 0xF, false));
}
// sum inside each row of 16 lanes; every lane of a row receives its row's sum
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]: lane ^ 1
  v += dpp_f<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]: lane ^ 2
  v += dpp_f<0x141, 0xF>(v);   // row_half_mirror: the other quad of each 8
  v += dpp_f<0x140, 0xF>(v);   // row_mirror: the other half of the row
  return v;
}
template <> __device__ __forceinline__ float wave_sum<float>(float v) {
  v = row16_sum(v);
  v += dpp_f<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3: rows 0+1, rows 2+3
  v += dpp_f<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3: row 3 now holds the total
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
// fp64, the same way in two halves
template <int CTRL, int ROW_MASK> __device__ __forceinline__ double dpp_d(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_d<0xB1, 0xF>(v);
  v += dpp_d<0x4E, 0xF>(v);
  v += dpp_d<0x141, 0xF>(v);
  v += dpp_d<0x140, 0xF>(v);
  return v;
}
template <> __device__ __forceinline__ double wave_sum<double>(double v) {
  v = row16_sum(v);
  v += dpp_d<0x142, 0xA>(v);
  v += dpp_d<0x143, 0xC>(v);
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// v^-1/2 to the last bit of fp32 or nearly so: the hardware's estimate (about 2^-23) and one Newton step in fp64 (1e-13);
// outside the estimate's range - variances that vanish, infinities - the library's square root.
__device__ __forceinline__ float inv_sqrt(double v) {
  const float x = (float)v;
  if (x > 1e-30f && x < 1e30f) {
    const double r = (double)__builtin_amdgcn_rsqf(x);
    return (float)(r * (1.5 - 0.5 * v * r * r));
  }
  return (float)(1.0 / sqrt(v));
}

// ---------------------------------------------------------------------------------------------
// Column sums from per-group partial sums, colpart [groups][nwhich][N]: 64 consecutive columns per workgroup (coalesced), the
// groups dealt over its SL wavefronts, loads in flight per thread by the eight (the phase is pure latency: a few tens of MB), fp64
// sums in a fixed order.
template <class C, int SL = 16>
__device__ __forceinline__ void b2_columns(int64_t N, int groups, int nwhich, const C* __restrict__ colpart, int cblock,
                                           int which, float* __restrict__ out, double (*red)[64]) {
  constexpr int kLoads = SL >= 16 ? 8 : 16;
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int64_t col = (int64_t)cblock * 64 + lane;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  if (col < N) {
    const C* src = colpart + (int64_t)which * N + col;
    const int64_t gstride = (int64_t)nwhich * N;
    int g = slice;
    for (; g + (kLoads - 1) * SL < groups; g += kLoads * SL) {
      C v[kLoads];
#pragma unroll
      for (int e = 0; e < kLoads; e++) v[e] = src[(int64_t)(g + e * SL) * gstride];
#pragma unroll
      for (int e = 0; e < kLoads; e++) a[e & 3] += (double)v[e];
    }
#pragma unroll 4
    for (; g < groups; g += SL) a[0] += (double)src[(int64_t)g * gstride];
  }
  red[slice][lane] = (a[0] + a[1]) + (a[2] + a[3]);
  __syncthreads();
  if (slice == 0 && col < N) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < SL; w++) t += red[w][lane];
    out[col] = (float)t;
  }
}

}  // namespace fdl
