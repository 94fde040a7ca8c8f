// C-ABI entry points of libfdl: argument validation, launch plan / workspace layout, and the sequence of
// kernel launches for the forward and backward pass of the fused dense-layer block.
#include "../../include/fdl.h"
#include "internal.h"

#include <cmath>
#include <cstdio>
#include <mutex>

namespace fdl {
namespace {

constexpr int64_t kMaxDim = (int64_t)1 << 24;       // per dimension
constexpr int64_t kMaxElems = (int64_t)1 << 40;     // per matrix

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

__global__ void zero_f32_kernel(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0.0f;
}
__global__ void zero_u16_kernel(unsigned short* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

bool shape_ok(int64_t M, int64_t K, int64_t N) {
  if (M < 0 || K < 1 || N < 1) return false;
  if (M > kMaxDim || K > kMaxDim || N > kMaxDim) return false;
  if (M * N > kMaxElems || M * K > kMaxElems || N * K > kMaxElems) return false;
  return true;
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// fp32 storage: all tiles as they are, where there is no scratch for the sums of split ones
F64Split f64_unsplit(int64_t I, int64_t J, int64_t R) { return F64Split{((I + 63) / 64) * ((J + 63) / 64), 0, 1, f64_plan(I, J, R).small}; }

// room for the sums of split reductions in 128 x 128 tiles; kept: what the other kernels' plan holds in their place
constexpr size_t kMidMostSums = (size_t)64 << 20;
size_t mid_room(Room room, size_t kept) { return room == Room::kAll ? (kept > kMidMostSums ? kept : kMidMostSums) : (room == Room::kTight ? kept : 0); }

// Estimated time, us, of dX and dW on the kernels of q, with their copies and sums of split reductions: prices fitted together with
// mid_grads_cost's to whole backward passes of 1300 shapes (see make_grad_plan for what the rule loses).
double grads_cost(const GradPlan& q) {
  const int64_t Np = q.pad ? fast_pad_dim(q.N) : q.N, Kp = q.pad ? fast_pad_dim(q.K) : q.K, Mp = q.M > 0 ? q.M : 1;
  const double mk = (double)Mp * (double)q.K / 1e6, nk = (double)q.N * (double)q.K / 1e6;
  auto rounds = [](int64_t tiles) { return (double)((tiles + 255) / 256); };
  auto tiles = [](int64_t I, int64_t J) { return ((I + 255) / 256) * ((J + 255) / 256); };
  double cost = 0.0;
  if (q.pad) cost += 5.4 + ((double)(Np * Kp) + (q.stage_x ? (double)(Mp * Kp) : 0.0)) * 2.0 / 1e6 * 0.27;
  if (q.pair) {
    const int64_t a = Np / q.split_a, b = q.b4_fast_rows / q.split_b;
    cost += 11.7 + (double)(a > b ? a : b) * 0.0137;
    if (q.split_a > 1) cost += q.split_a * mk * 1.05;
  } else {
    cost += q.b3_fast ? 11.7 + rounds(tiles(Kp, Mp)) * ((double)Np * 0.0145 + 1.3) : 1.2 * generic_xwt_cost(Mp, q.N, q.K);
    cost += q.b4_fast ? 11.7 + rounds(tiles(Kp, q.N) * q.split_b) * ((double)q.b4_fast_rows / q.split_b * 0.0137 + 1.3)
                      : 1.2 * generic_xwt_cost(q.N, Mp, q.K);
  }
  if (q.extra) cost += 1.2 * generic_xwt_cost(q.N, Mp - q.b4_fast_rows, q.K);
  if (q.parts_b > 1) cost += q.parts_b * nk * 1.05;
  return cost;
}

thread_local bool t_failure_noted = false;

}  // namespace

void note_failure(const char* what, hipError_t e) {
  fprintf(stderr, "libfdl: %s failed: %s\n", what, hipGetErrorString(e));
  t_failure_noted = true;
}

bool device_info(DeviceInfo* out) {
  static std::mutex mu;
  static DeviceInfo cache[kMaxDevices];
  static bool have[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) { note_failure("hipGetDevice", e); return false; }
  if (dev < 0 || dev >= kMaxDevices) { note_failure("device ordinal beyond the supported range", hipErrorInvalidDevice); return false; }
  std::lock_guard<std::mutex> lock(mu);
  if (!have[dev]) {
    int cus = 0, xcds = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess || cus < 1) { note_failure("hipDeviceGetAttribute(compute units)", e); return false; }
    // a runtime that does not know the attribute yet reports an error: every gfx950 part has 8 dies
    if (hipDeviceGetAttribute(&xcds, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess || xcds < 1) {
      (void)hipGetLastError();
      xcds = 8;
    }
    if (cus % xcds != 0) xcds = 1;
    cache[dev].cus = cus; cache[dev].xcds = xcds;
    have[dev] = true;
  }
  *out = cache[dev];
  return true;
}

bool ensure_dynamic_lds(const void* kernel, int bytes, OnceFlags* flags) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) { note_failure("hipGetDevice", e); return false; }
  if (flags->done[dev].load(std::memory_order_acquire)) return true;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);   // idempotent: a race is harmless
  if (e != hipSuccess) { note_failure("hipFuncSetAttribute(dynamic LDS size)", e); return false; }
  flags->done[dev].store(1, std::memory_order_release);
  return true;
}

static void tight_pitch(GradPlan* q);

bool make_plan(int dt, int64_t M, int64_t K, int64_t N, Room room, Plan* p, bool forward_only) {
  if (dt != kF32 && dt != kBF16) return false;
  if (!shape_ok(M, K, N)) return false;
  const size_t cs = dt == kF32 ? 8 : 4;   // arithmetic element
  const bool split = room == Room::kAll || room == Room::kTight;
  Plan q = {};
  q.dt = dt; q.M = M; q.K = K; q.N = N;

  // ---- which contraction kernels run
  // bf16, forward: the kernel with the lowest estimated time.  The tiled one runs where N and K are multiples of the tile and
  // the pipeline round (as they are), or - padded mode - on N and K rounded up to the tile, on zero-padded copies of the weights
  // (and of X where its rows start at any element), leaving the surplus unstored.
  const bool can_pad = dt == kBF16 && fast_padded_supported(M, K, N), can_tile = dt == kBF16 && fast_f1_supported(M, K, N);
  const int64_t Np = can_pad ? fast_pad_dim(N) : N, Kp = can_pad ? fast_pad_dim(K) : K;
  const int64_t Mp = M > 0 ? M : 1;

  // ---- forward
  double f1_cost = 0.0;
  const Xwt f1 = dt == kBF16 ? pick_xwt(Mp, K, N, room != Room::kNoCopies, true, false, &f1_cost) : Xwt::kGeneric;
  const bool tiled = f1 == Xwt::kTiled || f1 == Xwt::kPadded;
  q.f1_skinny = f1 == Xwt::kSkinny;
  q.pad = f1 == Xwt::kPadded;
  q.stage_x = q.pad && fast_padded_stages_x(K);
  q.f1_fast = tiled;
  q.f1_wb = generic_wb(Mp, N);
  size_t off = 0;
  q.off_rows = off; off += align256(f2_part_bytes(dt, Mp, N));
  q.off_xtail = off; off += align256(!tiled ? 0 : (q.pad ? fast_padded_x_bytes(M, K, q.stage_x != 0) : fast_f1_tail_bytes(M, K)));
  q.off_wpad_f = off; off += align256(tiled && q.pad ? (size_t)Np * Kp * 2 : 0);
  q.off_bpad_f = off; off += align256(tiled && q.pad ? (size_t)Np * 4 : 0);
  if (dt == kF32) q.f1_s64 = split ? f64_plan(Mp, N, K) : f64_unsplit(Mp, N, K);
  q.f1_split = tiled && split ? fast_xwt_split(M, K, N) : 1;
  q.off_part = off; off += align256(dt == kF32 ? f64_part_bytes(q.f1_s64) : fast_xwt_part_bytes(M, N, q.f1_split));
  q.fwd_bytes = off;
  // (128 x 128 tiles need no copies: the sums of their split reduction lie where those would)
  if (dt == kBF16 && mid_supported(Mp, K, N)) {
    int parts = 1;
    if (mid_margin(Mp) * mid_xwt_cost(Mp, K, N, mid_room(room, off - q.off_xtail), &parts) < f1_cost) {
      q.f1_mid = 1; q.f1_split = parts; q.off_part = q.off_xtail;
      const size_t need = q.off_part + align256(fast_xwt_part_bytes(Mp, N, parts));
      if (need > q.fwd_bytes) q.fwd_bytes = need;
    }
  }
  // The static entry point's limit is part of its contract (see the header) and does not move with the plan: the tiled
  // kernels' copies for whole 16-byte rows, and 8 bytes per (row, column tile) unless rows of whole vectors up to 8192 meet
  // the tiled kernel.
  const bool copies = can_pad && N % 8 == 0 && K % 8 == 0 && K >= 128;
  const bool limit_fast = copies || (!can_pad && can_tile);
  const int64_t limit_tile = limit_fast ? 128 : (dt == kF32 ? 32 : 16 * q.f1_wb);
  q.static_need = (limit_fast && N % 8 == 0 && N <= 8192 ? 0 : align256((size_t)((N + limit_tile - 1) / limit_tile) * Mp * 8)) +
                  align256(copies ? fast_padded_tail_bytes(K) : (limit_fast ? fast_f1_tail_bytes(M, K) : 0)) +
                  align256(copies ? (size_t)Np * Kp * 2 : 0) + align256(copies ? (size_t)Np * 4 : 0);
  if (forward_only) { *p = q; return true; }

  // ---- backward
  // dZ in 32 x 32 blocks where only the fused row kernel writes it and only the tuned kernels read it; the vector path of
  // the row kernel needs N % 8 = 0, which the tiles imply
  // (the row kernel pays for it with about 8 % of its time where a row fills 1024 threads, dX gains about 9 %: not
  //  worth it when such rows meet a short K)
  q.b1_fused = b1_fused_supported(dt, N, Np);
  const bool may_block = q.b1_fused && (K >= 1024 || N <= 4096);
  if (q.b1_fused) {
    const int64_t want = b1_fused_groups(dt, Mp, N);
    q.b1_groups = (int)(Mp < want ? Mp : want);
    q.b1_rows_per_group = 0;
  } else {
    const int64_t rpg = b1b_rows_per_group(dt, Mp, N);
    q.b1_rows_per_group = (int)rpg;
    q.b1_groups = (int)((Mp + rpg - 1) / rpg);
  }
  off = 0;
  q.off_c12 = off; off += align256(q.b1_fused ? 0 : (size_t)2 * Mp * cs);
  q.off_colpart = off; off += align256((size_t)q.b1_groups * 3 * N * cs);
  make_grad_plan(dt, M, K, N, room, may_block, &off, &q.g);
  tight_pitch(&q.g);
  if (q.b1_fused) {      // (the partials' room is that of a row per group)
    const int64_t slots = b1_fused_slots(dt, N, q.g.ldz), most = (Mp + slots - 1) / slots;
    if (q.b1_groups > most) q.b1_groups = (int)most;
  }
  q.bwd_bytes = off;
  // (one buffer for both passes and for fdl_forward_inference, which keeps mean and rstd in it)
  const size_t fwd_all = q.fwd_bytes + 2 * align256((size_t)Mp * 4) + 256;
  q.bytes = fwd_all > q.bwd_bytes ? fwd_all : q.bwd_bytes;
  *p = q;
  return true;
}

// The two contractions that end a backward pass, dX [M,K] = dZ W and dW [N,K] = dZ^T X, with the workspace regions they
// need behind *off.  may_block: the kernel that writes dZ can write it in 32 x 32 blocks.
void make_grad_plan(int dt, int64_t M, int64_t K, int64_t N, Room room, bool may_block, size_t* off, GradPlan* p) {
  const bool split = room == Room::kAll || room == Room::kTight;
  GradPlan q = {};
  const size_t ts = dt == kF32 ? 4 : 2;
  const int64_t Mp = M > 0 ? M : 1;
  q.dt = dt; q.M = M; q.K = K; q.N = N;
  q.pad = dt == kBF16 && fast_padded_supported(M, K, N);
  q.stage_x = q.pad && fast_padded_stages_x(K);
  const int64_t Np = q.pad ? fast_pad_dim(N) : N, Kp = q.pad ? fast_pad_dim(K) : K;
  q.ldz = Np;
  q.b3_fast = q.pad || (dt == kBF16 && fast_b3_supported(M, K, N));
  q.b3_wb = generic_wb(Mp, K);
  q.b4_wb = generic_wb(N, K);
  if (q.pad) {
    q.b4_fast_rows = fast_padded_b4_rows(M, K);
    q.b4_fast = q.b4_fast_rows >= 128;
    if (!q.b4_fast) q.b4_fast_rows = 0;
  } else {
    q.b4_fast = dt == kBF16 && fast_b4_supported(M, K, N);
    q.b4_fast_rows = q.b4_fast ? fast_b4_rows(M) : 0;
  }
  if (!split && q.b4_fast_rows < M) { q.b4_fast = 0; q.b4_fast_rows = 0; }   // (two partial sums: all of dW on the generic kernel)
  q.extra = q.b4_fast && q.b4_fast_rows < M ? 1 : 0;    // rows of dW's reduction left to the generic kernel: one more partial
  q.split_a = 1;
  q.split_b = q.b4_fast && split ? fast_b4_split(q.b4_fast_rows, K, N) : 1;
  q.pair = split && q.b3_fast && q.b4_fast && fast_pair_plan(M, K, N, q.b4_fast_rows, &q.split_a, &q.split_b);
  q.blocked = may_block && dt == kBF16 && !q.pad && q.b3_fast && q.b4_fast && q.b4_fast_rows == M && M % 32 == 0 && N % 32 == 0;
  // dZ: the fast dX kernel reads whole 256-row tiles, so the buffer is rounded up (the surplus rows never reach an output)
  q.off_dz = *off; *off += align256((size_t)fast_padded_rows(Mp) * Np * ts);
  // fp32 partial sums: the parts of a split reduction, one more for the rows the fast kernel leaves to the generic one
  q.parts_b = q.split_b + q.extra;
  q.off_dxpart = *off; *off += align256(q.split_a > 1 ? (size_t)q.split_a * partial_stride(M * K) * 4 : 0);
  q.off_dwpart = *off; *off += align256(q.parts_b > 1 ? (size_t)q.parts_b * partial_stride(N * K) * 4 : 0);
  const size_t sums = *off - q.off_dxpart;
  q.off_wpad = *off; *off += align256(q.pad ? (size_t)Np * Kp * 2 : 0);
  q.off_xpad = *off; *off += align256(q.stage_x ? fast_padded_x_bytes(M, K, true) : 0);
  if (dt == kF32) {
    q.s64_a = split ? f64_plan(Mp, K, N) : f64_unsplit(Mp, K, N);
    q.s64_b = split ? f64_plan(N, K, Mp) : f64_unsplit(N, K, Mp);
    q.s64_a.small = q.s64_b.small = f64_small_grads(Mp, K, N, split ? &q.s64_a : nullptr, &q.s64_b);
    q.off_part64_a = *off; *off += align256(f64_part_bytes(q.s64_a));
    q.off_part64_b = *off; *off += align256(f64_part_bytes(q.s64_b));
  }
  if (dt == kBF16 && mid_supported(Mp, K, N)) {
    int sa = 1, sb = 1;
    // 7 % for the estimates' spread.  4149 shapes (256 to 40000 rows), whole backward passes, both forced: the kernels picked take 1.008
    // times the faster ones' time on average, 1.045 at the 95th percentile, 1.25 at most, nearly always 256 x 256 tiles; 74 are more than
    // 2 % slower than in those (7.5 % at most).  (The prices were fitted before the 256 x 256 tiles took 16 x 16 x 32 MFMAs.)
    if (1.07 * mid_grads_cost(Mp, K, N, mid_room(room, sums), &sa, &sb) < grads_cost(q)) {
      q.mid = 1; q.blocked = 0; q.split_a = sa; q.split_b = q.parts_b = sb;
      const size_t na = align256(sa > 1 ? (size_t)sa * partial_stride(M * K) * 4 : 0), nb = align256(sb > 1 ? (size_t)sb * partial_stride(N * K) * 4 : 0);
      if (na + nb > sums) { q.off_dxpart = *off; *off += na + nb; }      // (the copies of padded mode stay where they are)
      q.off_dwpart = q.off_dxpart + na;
    }
  }
  *p = q;
}

// 128 x 128 tiles: dZ's pitch, where the buffer holds it.  Whole cache lines where those are at most an eighth longer than the row,
// else the smallest one whose rows are aligned vectors.  Whole backward passes of 3400 shapes whose N is no multiple of 64, lines
// against vectors: rows at most a tenth longer, from 10^7 elements of dZ on 4 % faster (16865 x 100 x 15555 1000 to 919 us, 20067 x
// 473 x 824 102 to 91), 1 - 2 % from 10^6 on, equal below; a fifth longer and more 1 - 5 % slower from 10^6 on.  Whole tiles of 256
// are never faster than lines.
static void tight_pitch(GradPlan* q) {
  if (!q->mid) return;
  const int64_t Mp = q->M > 0 ? q->M : 1, room = fast_padded_rows(Mp) * q->ldz, lines = (q->N + 63) / 64 * 64;
  const int64_t want = (lines - q->N) * 8 <= q->N && Mp * lines <= room ? lines : (q->N + 7) / 8 * 8;
  if (Mp * want <= room) q->ldz = want;
}

}  // namespace fdl

using namespace fdl;

extern "C" const char* fdl_status_string(fdl_status s) {
  switch (s) {
    case FDL_OK: return "FDL_OK";
    case FDL_ERR_NULL: return "FDL_ERR_NULL: a required pointer is NULL";
    case FDL_ERR_SHAPE: return "FDL_ERR_SHAPE: M, K or N out of the supported range";
    case FDL_ERR_DTYPE: return "FDL_ERR_DTYPE: unknown dtype";
    case FDL_ERR_EPS: return "FDL_ERR_EPS: eps must be finite and >= 0";
    case FDL_ERR_WORKSPACE: return "FDL_ERR_WORKSPACE: workspace missing or too small";
    case FDL_ERR_ALIGN: return "FDL_ERR_ALIGN: pointer not sufficiently aligned";
    case FDL_ERR_LAUNCH: return "FDL_ERR_LAUNCH: HIP reported a launch error";
  }
  return "unknown fdl_status";
}

extern "C" size_t fdl_workspace_bytes(fdl_dtype dt, int64_t M, int64_t K, int64_t N) {
  Plan p;
  if (!make_plan((int)dt, M, K, N, Room::kAll, &p)) return 0;
  return p.bytes;
}

// A workspace that lacks only the room for split reductions serves the call all the same, without them, and the forward
// products do without the operands' copies: needs fall with M where few rows make a reduction split or a larger batch runs on a
// kernel without copies, and a caller that allocated for its largest batch must not fail on a smaller one.
// make(room, plan) fills a plan (false: unsupported shape) with its need in plan->bytes.
template <class P, class Make> static fdl_status fit_plan(const void* workspace, size_t have, P* plan, Make make) {
  if (!make(Room::kAll, plan)) return FDL_ERR_SHAPE;
  if (workspace == nullptr) return FDL_ERR_WORKSPACE;
  for (Room room : {Room::kTight, Room::kNoSplit, Room::kNoCopies})
    if (have < plan->bytes) (void)make(room, plan);
  if (have < plan->bytes) return FDL_ERR_WORKSPACE;
  if (!aligned(workspace, 256)) return FDL_ERR_ALIGN;
  return FDL_OK;
}

static fdl_status check_common(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* workspace,
                               size_t workspace_bytes, Plan* p) {
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  return fit_plan(workspace, workspace_bytes, p, [&](Room room, Plan* q) { return make_plan((int)dt, M, K, N, room, q); });
}

// ---- optional per-phase event instrumentation
static hipEvent_t g_phase_events[2 * FDL_PHASE_COUNT];
static bool g_phase_events_on = false;

extern "C" fdl_status fdl_set_phase_events(void* const* events, int count) {
  if (events == nullptr) { g_phase_events_on = false; return FDL_OK; }
  if (count != 2 * FDL_PHASE_COUNT) return FDL_ERR_SHAPE;
  for (int i = 0; i < count; i++) {
    if (events[i] == nullptr) return FDL_ERR_NULL;
    g_phase_events[i] = static_cast<hipEvent_t>(events[i]);
  }
  g_phase_events_on = true;
  return FDL_OK;
}

namespace {
struct PhaseTimer {
  int phase; hipStream_t s;
  PhaseTimer(int p, hipStream_t st) : phase(p), s(st) {
    if (g_phase_events_on) (void)hipEventRecord(g_phase_events[2 * phase], s);
  }
  ~PhaseTimer() {
    if (g_phase_events_on) (void)hipEventRecord(g_phase_events[2 * phase + 1], s);
  }
};
}  // namespace

// The HIP "last error" is per-thread state shared with everything else the caller does on this thread (an
// allocator that probed and recovered from an out-of-memory condition leaves it set): it is cleared on entry so
// that only this call's launches are reported, and the reason of a failed launch goes to stderr.
static void clear_stale_error() { (void)hipGetLastError(); t_failure_noted = false; }
static fdl_status launch_status() {
  const hipError_t e = hipGetLastError();
  if (t_failure_noted) { t_failure_noted = false; return FDL_ERR_LAUNCH; }
  if (e == hipSuccess) return FDL_OK;
  fprintf(stderr, "libfdl: kernel launch failed: %s\n", hipGetErrorString(e));
  return FDL_ERR_LAUNCH;
}

// Validation shared by the forward entry points (everything except the scratch buffer).
static fdl_status check_forward_args(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* X, const void* W,
                                     const float* b, const float* gamma, const float* beta, float eps, const void* Y,
                                     const void* Zsave, const float* mean, const float* rstd, Plan* p) {
  if (!X || !W || !b || !gamma || !beta || !Y || !Zsave || !mean || !rstd) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  if (!(eps >= 0.0f) || std::isinf(eps)) return FDL_ERR_EPS;
  if (!make_plan((int)dt, M, K, N, Room::kAll, p)) return FDL_ERR_SHAPE;
  return FDL_OK;
}
static bool forward_args_aligned(const void* X, const void* W, const float* b, const float* gamma, const float* beta,
                                 const void* Y, const void* Zsave, const float* mean, const float* rstd) {
  return aligned(X, 16) && aligned(W, 16) && aligned(Y, 16) && aligned(Zsave, 16) && aligned(b, 16) &&
         aligned(gamma, 16) && aligned(beta, 16) && aligned(mean, 16) && aligned(rstd, 16);
}

// The launches of the forward pass; ws: at least p.fwd_bytes bytes of device scratch, 256-byte aligned.
static fdl_status forward_launches(const Plan& p, const void* X, const void* W, const float* b, const float* gamma,
                                   const float* beta, float eps, void* Y, void* Zsave, float* mean, float* rstd,
                                   char* ws, hipStream_t s) {
  const int64_t M = p.M, K = p.K, N = p.N;
  // fp32, few tiles, all split: the row kernel adds the parts up
  const bool sums = p.dt == kF32 && !p.f1_s64.small && p.f1_s64.split > 1 && p.f1_s64.whole == 0 && f2_takes_sums(N);
  F64Sums parts = {};
  {
    PhaseTimer t(FDL_PHASE_F1, s);
    if (p.f1_mid) {
      launch_mid_xwt(0, M, K, N, X, W, b, nullptr, Zsave, N, p.f1_split, ws + p.off_part, s);
    } else if (p.f1_skinny) {
      launch_skinny_xwt(0, M, K, N, X, W, b, nullptr, Zsave, N, s);
    } else if (p.pad) {
      void* Wp = ws + p.off_wpad_f;
      float* bp = reinterpret_cast<float*>(ws + p.off_bpad_f);
      StageJobs j = {};
      stage_padded(&j, M, K, N, p.stage_x != 0, X, W, b, ws + p.off_xtail, Wp, bp);
      launch_stage(j, s);
      launch_fast_xwt_padded(0, M, K, N, p.stage_x != 0, X, ws + p.off_xtail, Wp, bp, nullptr, Zsave, p.f1_split, ws + p.off_part, s);
    } else if (p.f1_fast) {
      launch_fast_xwt(0, M, K, N, X, false, W, b, nullptr, Zsave, false, ws + p.off_xtail, s, p.f1_split, ws + p.off_part);
    } else {
      GemmDesc g = {X, W, M, N, K, K, K, true, true, p.f1_wb};
      if (sums) parts = launch_f64_parts(g, p.f1_s64, b, Zsave, ws + p.off_part, s);
      else if (p.dt == kF32) launch_f64(0, g, p.f1_s64, b, nullptr, Zsave, ws + p.off_part, s);
      else launch_generic_xwt(0, g, b, nullptr, Zsave, N, s);
    }
  }
  {
    PhaseTimer t(FDL_PHASE_FS, s);   // (the statistics are F2's own: nothing is launched here)
  }
  {
    PhaseTimer t(FDL_PHASE_F2, s);
    if (sums) launch_f2_sums(M, N, eps, parts, gamma, beta, Y, mean, rstd, s);
    else launch_f2(p.dt, M, N, eps, Zsave, gamma, beta, Y, mean, rstd, ws + p.off_rows, s);
  }
  return launch_status();
}

extern "C" fdl_status fdl_forward(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* X, const void* W,
                                  const float* b, const float* gamma, const float* beta, float eps, void* Y,
                                  void* Zsave, float* mean, float* rstd, void* workspace, size_t workspace_bytes,
                                  void* hip_stream) {
  Plan p;
  fdl_status st = check_forward_args(dt, M, K, N, X, W, b, gamma, beta, eps, Y, Zsave, mean, rstd, &p);
  if (st != FDL_OK) return st;
  st = check_common(dt, M, K, N, workspace, workspace_bytes, &p);
  if (st != FDL_OK) return st;
  if (!forward_args_aligned(X, W, b, gamma, beta, Y, Zsave, mean, rstd)) return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  return forward_launches(p, X, W, b, gamma, beta, eps, Y, Zsave, mean, rstd, static_cast<char*>(workspace),
                          static_cast<hipStream_t>(hip_stream));
}

// ---- forward pass on the library's own scratch: no allocation, no workspace argument ----------------------------
// The scratch lives in device memory that belongs to the loaded code object: one copy per GPU, present from the
// moment the library is loaded on that GPU until the process ends.  In host code the array's name is only a handle;
// its device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[FDL_STATIC_SCRATCH_BYTES];

static char* static_scratch_address() {
  static std::mutex mu;
  static char* ptr[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) { note_failure("hipGetDevice", e); return nullptr; }
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess || a == nullptr) { note_failure("hipGetSymbolAddress(static scratch)", e); return nullptr; }
    ptr[dev] = static_cast<char*>(a);
  }
  return ptr[dev];
}

extern "C" fdl_status fdl_forward_static(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* X, const void* W,
                                         const float* b, const float* gamma, const float* beta, float eps, void* Y,
                                         void* Zsave, float* mean, float* rstd, void* hip_stream) {
  Plan p;
  const fdl_status st = check_forward_args(dt, M, K, N, X, W, b, gamma, beta, eps, Y, Zsave, mean, rstd, &p);
  if (st != FDL_OK) return st;
  if (p.static_need > (size_t)FDL_STATIC_SCRATCH_BYTES) return FDL_ERR_WORKSPACE;   // more than the array is stated to hold
  if (p.f1_mid) {     // (needs no copies; no room for the sums of a split reduction: unsplit)
    if (p.off_part + fast_xwt_part_bytes(M, N, p.f1_split) > (size_t)FDL_STATIC_SCRATCH_BYTES) p.f1_split = 1;
    p.fwd_bytes = p.off_part;
  }
  if (p.fwd_bytes > (size_t)FDL_STATIC_SCRATCH_BYTES && p.f1_split > 1) {
    p.f1_split = 1; p.fwd_bytes = p.off_part;         // (the sums of a split reduction are the last region here)
  }
  if (p.fwd_bytes > (size_t)FDL_STATIC_SCRATCH_BYTES && p.pad && p.stage_x && !p.f1_skinny && fast_padded_can_skip_copy(K)) {
    // X as it is: only its last row tile is copied
    p.stage_x = 0;
    p.off_wpad_f = p.off_xtail + align256(fast_padded_x_bytes(M, K, false));
    p.off_bpad_f = p.off_wpad_f + align256((size_t)fast_pad_dim(N) * fast_pad_dim(K) * 2);
    p.fwd_bytes = p.off_bpad_f + align256((size_t)fast_pad_dim(N) * 4);
  }
  if (p.fwd_bytes > (size_t)FDL_STATIC_SCRATCH_BYTES) {
    p.pad = 0; p.f1_fast = 0; p.fwd_bytes = p.off_xtail;   // no room for the padded copies either: the generic kernel needs none,
    p.f1_s64 = f64_unsplit(M, N, K);                   // nor the fp64 kernel, with all tiles whole
  }
  if (!forward_args_aligned(X, W, b, gamma, beta, Y, Zsave, mean, rstd)) return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  char* ws = static_scratch_address();
  if (ws == nullptr) return launch_status();
  // every scratch location a forward pass reads has been written earlier in the same pass (padded
  // weights, the padded copy of X's last rows), so nothing has to be cleared between calls
  return forward_launches(p, X, W, b, gamma, beta, eps, Y, Zsave, mean, rstd, ws, static_cast<hipStream_t>(hip_stream));
}

// ---- dX and dW (see make_grad_plan) ---------------------------------------------------------------------------------
// whether the contractions leave fp32 partial sums behind for launch_finish
static bool grad_leaves_sums(const GradPlan& p) { return p.split_a > 1 || p.parts_b > 1; }

// padded mode: the copies the contractions read, and zeros in the rows behind dZ's last where dW's reduction covers them
static void stage_grad(const GradPlan& p, StageJobs* j, const void* X, const void* W, char* ws) {
  stage_padded(j, p.M, p.K, p.N, true, p.stage_x ? X : nullptr, W, nullptr, ws + p.off_xpad, ws + p.off_wpad, nullptr);
  if (p.b4_fast_rows > p.M)
    stage_matrix(j, nullptr, 0, 0, 0, ws + p.off_dz + (size_t)p.M * p.ldz * 2, p.b4_fast_rows - p.M, p.ldz);
}

static void sum_later(TailSums* tj, int k, const void* part, int parts, int64_t n, void* out) {
  tj->part[k] = static_cast<const float*>(part); tj->parts[k] = parts; tj->n[k] = n; tj->out[k] = out;
}

// fp32 storage: the operands of the launch that both contractions share
static F64Grads grad_f64(const GradPlan& p, const void* dZ, const void* W, const void* X, void* dX, void* dW, char* ws) {
  F64Grads a = {};
  a.dx = {dZ, W, p.M, p.K, p.N, p.ldz, p.K, true, false, 2};
  a.dw = {dZ, X, p.N, p.K, p.M, p.ldz, p.K, false, false, 2};
  a.qx = p.s64_a; a.qw = p.s64_b;
  a.dX = dX; a.partx = ws + p.off_part64_a; a.dW = dW; a.partw = ws + p.off_part64_b;
  return a;
}

// bf16 storage: dX = dZ W; where both contractions share a launch (p.mid, p.pair), dW too
static void launch_grad_dx(const GradPlan& p, const void* dZ, const void* W, const void* X, void* dX, void* dW, char* ws,
                           TailSums* tj, hipStream_t s) {
  const int64_t M = p.M, K = p.K, N = p.N;
  const int64_t Kp = p.pad ? fast_pad_dim(K) : K;
  if (p.mid) {
    MidGrads a = {};
    a.M = M; a.K = K; a.N = N; a.sa = p.split_a; a.sb = p.split_b;
    a.dZ = dZ; a.ldz = p.ldz; a.W = W; a.X = X;
    a.dX = dX; a.dxpart = ws + p.off_dxpart; a.dW = dW; a.dwpart = ws + p.off_dwpart;
    a.cols = *tj;
    launch_mid_grads(a, s);
    if (p.split_a > 1) sum_later(tj, 0, a.dxpart, p.split_a, M * K, dX);
    if (p.split_b > 1) sum_later(tj, 1, a.dwpart, p.split_b, N * K, dW);
  } else if (p.pair) {
    PairArgs a = {};
    a.M = M; a.K = K; a.N = N; a.rows = p.b4_fast_rows; a.sa = p.split_a; a.sb = p.split_b; a.extra = p.extra;
    a.dZ = dZ; a.ldz = p.ldz; a.dz_blocked = p.blocked != 0;
    a.W = p.pad ? ws + p.off_wpad : W; a.ldw = Kp;
    a.X = p.stage_x ? ws + p.off_xpad : X; a.ldx = p.stage_x ? Kp : K;
    a.dX = dX; a.dxpart = ws + p.off_dxpart; a.dW = dW; a.dwpart = ws + p.off_dwpart;
    launch_fast_pair(a, s);
    if (p.split_a > 1) sum_later(tj, 0, ws + p.off_dxpart, p.split_a, M * K, dX);
  } else if (p.pad) {
    launch_fast_b3_padded(M, K, N, dZ, ws + p.off_wpad, dX, s);
  } else if (p.b3_fast) {
    launch_fast_b3(M, K, N, dZ, p.blocked != 0, W, dX, s);
  } else {
    GemmDesc g = {dZ, W, M, K, N, p.ldz, K, true, false, p.b3_wb};
    launch_generic_store(g, dX, s);
  }
}

// dW = dZ^T X.  The fast kernel reduces over the first b4_fast_rows rows (a whole number of pipeline rounds); the few rows
// after them go through the generic kernel into one more fp32 partial sum.
static void launch_grad_dw(const GradPlan& p, const void* dZ, const void* X, void* dW, char* ws, TailSums* tj, hipStream_t s) {
  const int64_t K = p.K, N = p.N, Mf = p.b4_fast_rows;
  float* dwpart = reinterpret_cast<float*>(ws + p.off_dwpart);
  if (p.mid) return;       // (with dX)
  if (!p.b4_fast) {
    GemmDesc g = {dZ, X, N, K, p.M, p.ldz, K, false, false, p.b4_wb};
    launch_generic_store(g, dW, s);
    return;
  }
  if (p.pair) {
    // (with dX)
  } else if (p.pad) {
    launch_fast_b4_padded(Mf, K, N, p.split_b, p.extra, dZ, p.stage_x ? ws + p.off_xpad : X, p.stage_x ? fast_pad_dim(K) : K, dW,
                          dwpart, s);
  } else {
    launch_fast_b4(Mf, K, N, p.split_b, p.extra, dZ, p.blocked != 0, X, dW, dwpart, s);
  }
  if (p.extra) {
    const char* dZt = static_cast<const char*>(dZ) + (size_t)Mf * p.ldz * 2;
    const char* Xt = static_cast<const char*>(X) + (size_t)Mf * K * 2;
    GemmDesc g = {dZt, Xt, N, K, p.M - Mf, p.ldz, K, false, false, p.b4_wb};
    launch_generic_store_f32(g, dwpart + (size_t)p.split_b * partial_stride(N * K), s);
  }
  if (p.parts_b > 1) sum_later(tj, 1, dwpart, p.parts_b, N * K, dW);
}

extern "C" fdl_status fdl_backward(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* dY, const void* X,
                                   const void* W, const float* gamma, const void* Zsave, const float* mean,
                                   const float* rstd, void* dX, void* dW, float* db, float* dgamma, float* dbeta,
                                   void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!dY || !X || !W || !gamma || !Zsave || !mean || !rstd || !dX || !dW || !db || !dgamma || !dbeta)
    return FDL_ERR_NULL;
  Plan p;
  const fdl_status st = check_common(dt, M, K, N, workspace, workspace_bytes, &p);
  if (st != FDL_OK) return st;
  if (!aligned(dY, 16) || !aligned(X, 16) || !aligned(W, 16) || !aligned(Zsave, 16) || !aligned(dX, 16) ||
      !aligned(dW, 16) || !aligned(gamma, 16) || !aligned(mean, 16) || !aligned(rstd, 16) || !aligned(db, 16) ||
      !aligned(dgamma, 16) || !aligned(dbeta, 16))
    return FDL_ERR_ALIGN;
  clear_stale_error();
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (M == 0) {
    // no rows: every sum over rows is empty
    const int64_t nk = N * K;
    if (dt == FDL_F32) hipLaunchKernelGGL(zero_f32_kernel, dim3(256), dim3(256), 0, s, (float*)dW, nk);
    else hipLaunchKernelGGL(zero_u16_kernel, dim3(256), dim3(256), 0, s, (unsigned short*)dW, nk);
    hipLaunchKernelGGL(zero_f32_kernel, dim3(8), dim3(256), 0, s, db, N);
    hipLaunchKernelGGL(zero_f32_kernel, dim3(8), dim3(256), 0, s, dgamma, N);
    hipLaunchKernelGGL(zero_f32_kernel, dim3(8), dim3(256), 0, s, dbeta, N);
    return launch_status();
  }
  char* ws = static_cast<char*>(workspace);
  void* dZ = ws + p.g.off_dz;
  void* c12 = ws + p.off_c12;
  void* colpart = ws + p.off_colpart;

  {
    PhaseTimer t(FDL_PHASE_B1, s);
    if (p.b1_fused) {
      launch_b1_fused((int)dt, M, N, p.g.ldz, p.b1_groups, p.g.blocked != 0, dY, Zsave, gamma, mean, rstd, dZ, colpart, s);
    } else {
      launch_b1a((int)dt, M, N, dY, Zsave, gamma, mean, rstd, c12, s);
      launch_b1b((int)dt, M, N, p.g.ldz, p.b1_rows_per_group, p.b1_groups, dY, Zsave, gamma, mean, rstd, c12, dZ, colpart, s);
      if (p.g.pad && !p.g.mid) launch_zero_cols_bf16(dZ, M, N, p.g.ldz, s);   // the surplus columns enter the contractions
    }
  }
  // Where the contractions below leave split reductions behind (bf16 tuned path), their sums and the column sums
  // share one launch at the end of the pass; otherwise the column sums are finished here, or with both gradients in 128 x 128 tiles.
  const bool tail = grad_leaves_sums(p.g);
  TailSums tj = {};
  tj.colpart = static_cast<const float*>(colpart); tj.groups = p.b1_groups; tj.N = N; tj.kinds = 3;
  tj.col_out[0] = dbeta; tj.col_out[1] = dgamma; tj.col_out[2] = db;
  if (dt == FDL_F32) {
    const F64Grads a = grad_f64(p.g, dZ, W, X, dX, dW, ws);
    { PhaseTimer t(FDL_PHASE_B2, s); }      // (the column sums are finished with the contractions')
    { PhaseTimer t(FDL_PHASE_B3, s); launch_f64_grads(a, tj, s); }
    { PhaseTimer t(FDL_PHASE_B4, s); launch_f64_grads_finish(a, tj, s); }
    return launch_status();
  }
  {
    PhaseTimer t(FDL_PHASE_B2, s);
    if (!tail && !p.g.mid) launch_b2(N, p.b1_groups, colpart, dbeta, dgamma, db, s);
  }
  {
    PhaseTimer t(FDL_PHASE_B3, s);
    if (p.g.pad && !p.g.mid) {
      StageJobs j = {};
      stage_grad(p.g, &j, X, W, ws);
      launch_stage(j, s);
    }
    launch_grad_dx(p.g, dZ, W, X, dX, dW, ws, &tj, s);
  }
  {
    PhaseTimer t(FDL_PHASE_B4, s);
    launch_grad_dw(p.g, dZ, X, dW, ws, &tj, s);
    if (tail) launch_finish(tj, s);
  }
  return launch_status();
}


// =====================================================================================================================
// Forward-only variant and the sibling operators on the same kernels
// =====================================================================================================================

// ---- forward for inference: nothing is saved for a backward pass ---------------------------------------------------
// The pre-activation is written into Y and normalised there (the normalisation reads an element before it writes it),
// so no M x N scratch is needed: the workspace holds the row statistics and what the forward pass needs.
namespace {
struct InferencePlan { Plan p; size_t off_mean, off_rstd, bytes; };
bool make_inference_plan(int dt, int64_t M, int64_t K, int64_t N, Room room, InferencePlan* q) {
  if (!make_plan(dt, M, K, N, room, &q->p, /*forward_only=*/true)) return false;
  const int64_t Mp = M > 0 ? M : 1;
  size_t off = q->p.fwd_bytes;
  q->off_mean = off; off += align256((size_t)Mp * 4);
  q->off_rstd = off; off += align256((size_t)Mp * 4);
  q->bytes = off;
  return true;
}
}  // namespace

extern "C" size_t fdl_forward_inference_workspace_bytes(fdl_dtype dt, int64_t M, int64_t K, int64_t N) {
  InferencePlan q;
  if (!make_inference_plan((int)dt, M, K, N, Room::kAll, &q)) return 0;
  return q.bytes;
}

extern "C" fdl_status fdl_forward_inference(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* X, const void* W,
                                            const float* b, const float* gamma, const float* beta, float eps, void* Y,
                                            void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!X || !W || !b || !gamma || !beta || !Y) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  if (!(eps >= 0.0f) || std::isinf(eps)) return FDL_ERR_EPS;
  InferencePlan q;
  const fdl_status st = fit_plan(workspace, workspace_bytes, &q,
                                 [&](Room room, InferencePlan* p) { return make_inference_plan((int)dt, M, K, N, room, p); });
  if (st != FDL_OK) return st;
  if (!aligned(X, 16) || !aligned(W, 16) || !aligned(Y, 16) || !aligned(b, 16) || !aligned(gamma, 16) || !aligned(beta, 16))
    return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  char* ws = static_cast<char*>(workspace);
  return forward_launches(q.p, X, W, b, gamma, beta, eps, Y, /*Zsave=*/Y, reinterpret_cast<float*>(ws + q.off_mean),
                          reinterpret_cast<float*>(ws + q.off_rstd), ws, static_cast<hipStream_t>(hip_stream));
}

// ---- Linear + ReLU -------------------------------------------------------------------------------------------------
namespace {
// Workspace of the Linear+ReLU pair (one layout for both passes): the first-stage column partials of db, the copies the
// forward product needs (padded weights and bias, X or its last rows), and what the two gradient
// contractions need, the masked upstream gradient G among it (the dZ of GradPlan).
struct ReluPlan {
  int f1_mid;              // the forward product (and its recomputation) in 128 x 128 tiles, f1_split parts
  int f1_skinny;           // few rows: the forward product (and its recomputation) on the kernel made for them
  int f1_fast, f1_wb;      // the tuned kernel, on the operands as they are
  int pad;                 // or in padded mode (then the gradient contractions run in it too)
  GradPlan g;
  F64Split f1_s64;         // fp32 storage
  int f1_split;            // bf16, tiled: parts of the forward product's reduction
  size_t off_colpart, off_xtail, off_wpad, off_bpad, off_part, bytes;
};
bool make_relu_plan(int dt, int64_t M, int64_t K, int64_t N, Room room, ReluPlan* q) {
  const bool split = room == Room::kAll || room == Room::kTight;
  if (dt != kF32 && dt != kBF16) return false;
  if (!shape_ok(M, K, N)) return false;
  const size_t cs = dt == kF32 ? 8 : 4;
  const int64_t Mp = M > 0 ? M : 1;
  double f1_cost = 0.0;
  const Xwt f1 = dt == kBF16 ? pick_xwt(Mp, K, N, room != Room::kNoCopies, true, false, &f1_cost) : Xwt::kGeneric;
  const bool tiled = f1 == Xwt::kTiled || f1 == Xwt::kPadded;
  q->f1_split = tiled && split ? fast_xwt_split(M, K, N) : 1;
  const size_t kept = dt == kBF16 ? fast_xwt_part_bytes(M, N, q->f1_split) : 0;
  int parts = 1;
  q->f1_mid = dt == kBF16 && mid_supported(Mp, K, N) &&
              mid_margin(Mp) * mid_xwt_cost(Mp, K, N, mid_room(room, kept), &parts) < f1_cost;
  q->pad = f1 == Xwt::kPadded && !q->f1_mid;
  q->f1_skinny = f1 == Xwt::kSkinny;
  q->f1_fast = f1 == Xwt::kTiled && !q->f1_mid;
  q->f1_wb = generic_wb(Mp, N);
  size_t off = 0;
  q->off_colpart = off; off += align256((size_t)colsum_groups(Mp) * N * cs);
  // (the masking epilogue of the tuned forward product can write blocks)
  make_grad_plan(dt, M, K, N, room, /*may_block=*/q->f1_fast && q->f1_split == 1, &off, &q->g);
  if (!q->pad) tight_pitch(&q->g);       // (the padded product's masking epilogue writes whole tiles of columns)
  // the padded copies of W and (where all of it is copied) X serve the forward product and the gradient contractions
  q->off_wpad = q->g.off_wpad;
  q->off_xtail = q->g.off_xpad;
  // (the room of copies is kept where 128 x 128 tiles do without them: sizes do not depend on which of the kernels is picked)
  if (tiled && !q->g.stage_x) {
    q->off_xtail = off; off += align256(f1 == Xwt::kPadded ? fast_padded_tail_bytes(K) : fast_f1_tail_bytes(M, K));
  }
  q->off_bpad = off; off += align256(f1 == Xwt::kPadded ? (size_t)fast_pad_dim(N) * 4 : 0);
  if (dt == kF32) q->f1_s64 = split ? f64_plan(Mp, N, K) : f64_unsplit(Mp, N, K);
  if (q->f1_mid) q->f1_split = parts;
  const size_t sums = dt == kF32 ? f64_part_bytes(q->f1_s64) : fast_xwt_part_bytes(M, N, q->f1_split);
  q->off_part = off; off += align256(sums > kept ? sums : kept);
  q->bytes = off;
  return true;
}

// out = f(X W^T + b): kind 1 the forward output, 2 the masked upstream gradient (out: the G buffer of the plan).  In padded
// mode the operands' copies must have been staged (off_xtail, off_wpad, off_bpad).
void relu_product(const ReluPlan& q, int kind, int dt, int64_t M, int64_t K, int64_t N, const void* X, const void* W,
                  const float* b, const void* aux, void* out, char* ws, hipStream_t s) {
  if (q.f1_mid) {
    launch_mid_xwt(kind, M, K, N, X, W, b, aux, out, kind == 2 ? q.g.ldz : N, q.f1_split, ws + q.off_part, s);
  } else if (q.f1_skinny) {
    launch_skinny_xwt(kind, M, K, N, X, W, b, aux, out, kind == 2 ? q.g.ldz : N, s);
  } else if (q.pad) {
    launch_fast_xwt_padded(kind, M, K, N, q.g.stage_x != 0, X, ws + q.off_xtail, ws + q.off_wpad, reinterpret_cast<const float*>(ws + q.off_bpad),
                           aux, out, q.f1_split, ws + q.off_part, s);
  } else if (q.f1_fast) {
    launch_fast_xwt(kind, M, K, N, X, false, W, b, aux, out, kind == 2 && q.g.blocked != 0, ws + q.off_xtail, s, q.f1_split,
                    ws + q.off_part);
  } else {
    GemmDesc g = {X, W, M, N, K, K, K, true, true, q.f1_wb};
    if (dt == kF32) launch_f64(kind, g, q.f1_s64, b, aux, out, ws + q.off_part, s);
    else launch_generic_xwt(kind, g, b, aux, out, kind == 2 ? q.g.ldz : N, s);
  }
}
}  // namespace

extern "C" size_t fdl_linear_relu_workspace_bytes(fdl_dtype dt, int64_t M, int64_t K, int64_t N) {
  ReluPlan q;
  if (!make_relu_plan((int)dt, M, K, N, Room::kAll, &q)) return 0;
  return q.bytes;
}

extern "C" fdl_status fdl_linear_relu_forward(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* X, const void* W,
                                              const float* b, void* Y, void* workspace, size_t workspace_bytes,
                                              void* hip_stream) {
  if (!X || !W || !b || !Y) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  ReluPlan q;
  const fdl_status st = fit_plan(workspace, workspace_bytes, &q,
                                 [&](Room room, ReluPlan* p) { return make_relu_plan((int)dt, M, K, N, room, p); });
  if (st != FDL_OK) return st;
  if (!aligned(X, 16) || !aligned(W, 16) || !aligned(Y, 16) || !aligned(b, 16)) return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(workspace);
  if (q.pad) {
    StageJobs j = {};
    stage_padded(&j, M, K, N, q.g.stage_x != 0, X, W, b, ws + q.off_xtail, ws + q.off_wpad, reinterpret_cast<float*>(ws + q.off_bpad));
    launch_stage(j, s);
  }
  relu_product(q, 1, (int)dt, M, K, N, X, W, b, nullptr, Y, ws, s);
  return launch_status();
}

extern "C" fdl_status fdl_linear_relu_backward(fdl_dtype dt, int64_t M, int64_t K, int64_t N, const void* dY, const void* X,
                                               const void* W, const float* b, void* dX, void* dW, float* db,
                                               void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!dY || !X || !W || !b || !dX || !dW || !db) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  ReluPlan q;
  const fdl_status st = fit_plan(workspace, workspace_bytes, &q,
                                 [&](Room room, ReluPlan* p) { return make_relu_plan((int)dt, M, K, N, room, p); });
  if (st != FDL_OK) return st;
  if (!aligned(dY, 16) || !aligned(X, 16) || !aligned(W, 16) || !aligned(b, 16) || !aligned(dX, 16) || !aligned(dW, 16) ||
      !aligned(db, 16))
    return FDL_ERR_ALIGN;
  clear_stale_error();
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (M == 0) {
    const int64_t nk = N * K;
    if (dt == FDL_F32) hipLaunchKernelGGL(zero_f32_kernel, dim3(256), dim3(256), 0, s, (float*)dW, nk);
    else hipLaunchKernelGGL(zero_u16_kernel, dim3(256), dim3(256), 0, s, (unsigned short*)dW, nk);
    hipLaunchKernelGGL(zero_f32_kernel, dim3(8), dim3(256), 0, s, db, N);
    return launch_status();
  }
  char* ws = static_cast<char*>(workspace);
  void* G = ws + q.g.off_dz;
  void* colpart = ws + q.off_colpart;
  if (q.pad || (q.g.pad && !q.g.mid)) {
    // the copies serve the recomputation, where that is padded, and both gradient contractions, where those are
    StageJobs j = {};
    if (!q.pad) {
      stage_padded(&j, M, K, N, true, q.g.stage_x ? X : nullptr, W, nullptr, ws + q.g.off_xpad, ws + q.g.off_wpad, nullptr);
      // (the other kernels write columns up to N only: the surplus of G is cleared first, with the rows behind its last)
      stage_matrix(&j, nullptr, 0, 0, 0, G, q.g.b4_fast_rows > M ? q.g.b4_fast_rows : M, q.g.ldz);
    } else {
      stage_padded(&j, M, K, N, q.g.stage_x != 0, X, W, b, ws + q.off_xtail, ws + q.off_wpad, reinterpret_cast<float*>(ws + q.off_bpad));
      if (q.g.b4_fast_rows > M && !q.g.mid)
        stage_matrix(&j, nullptr, 0, 0, 0, static_cast<char*>(G) + (size_t)M * q.g.ldz * 2, q.g.b4_fast_rows - M, q.g.ldz);
    }
    launch_stage(j, s);
  }
  // G = dY where X W^T + b > 0: the pre-activation is recomputed and never stored
  relu_product(q, 2, (int)dt, M, K, N, X, W, b, dY, G, ws, s);
  launch_colsum_partial((int)dt, M, N, q.g.ldz, G, q.g.blocked != 0, colpart, s);
  // the column sums end with the contractions' split sums where those leave any, else here
  const bool tail = grad_leaves_sums(q.g);
  TailSums tj = {};
  tj.colpart = static_cast<const float*>(colpart); tj.groups = colsum_groups(M); tj.N = N; tj.kinds = 1; tj.col_out[0] = db;
  if (dt == FDL_F32) {
    const F64Grads a = grad_f64(q.g, G, W, X, dX, dW, ws);
    launch_f64_grads(a, tj, s);
    launch_f64_grads_finish(a, tj, s);
    return launch_status();
  }
  if (!tail && !q.g.mid) launch_colsum_finish(M, N, colpart, db, s);
  launch_grad_dx(q.g, G, W, X, dX, dW, ws, &tj, s);
  launch_grad_dw(q.g, G, X, dW, ws, &tj, s);
  if (tail) launch_finish(tj, s);
  return launch_status();
}

// ---- LayerNorm and RMSNorm forward ---------------------------------------------------------------------------------
static bool norm_shape_ok(int64_t M, int64_t N) {
  return M >= 0 && N >= 1 && M <= kMaxDim && N <= kMaxDim && M * N <= kMaxElems;
}

extern "C" fdl_status fdl_layernorm_forward(fdl_dtype dt, int64_t M, int64_t N, const void* A, const float* gamma,
                                            const float* beta, float eps, void* Y, float* mean, float* rstd,
                                            void* hip_stream) {
  if (!A || !gamma || !beta || !Y || !mean || !rstd) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  if (!(eps >= 0.0f) || std::isinf(eps)) return FDL_ERR_EPS;
  if (!norm_shape_ok(M, N)) return FDL_ERR_SHAPE;
  if (!aligned(A, 16) || !aligned(Y, 16) || !aligned(gamma, 16) || !aligned(beta, 16) || !aligned(mean, 16) || !aligned(rstd, 16))
    return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  launch_layernorm((int)dt, M, N, eps, A, gamma, beta, Y, mean, rstd, static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

extern "C" fdl_status fdl_rmsnorm_forward(fdl_dtype dt, int64_t M, int64_t N, const void* A, const float* weight, float eps,
                                          void* Y, void* hip_stream) {
  if (!A || !weight || !Y) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  if (!(eps >= 0.0f) || std::isinf(eps)) return FDL_ERR_EPS;
  if (!norm_shape_ok(M, N)) return FDL_ERR_SHAPE;
  if (!aligned(A, 16) || !aligned(Y, 16) || !aligned(weight, 16)) return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  launch_rmsnorm((int)dt, M, N, eps, A, weight, Y, static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

// ---- Llama feed-forward block, forward -----------------------------------------------------------------------------
namespace {
// Workspace: G and U [Mpad][H] in the storage type (the activation overwrites G; rows padded to whole tiles so that the
// down projection's fast kernel may read a partial last row tile; U only where the two products are separate kernels),
// then the padded copy of X's last rows.
struct FfnPlan {
  int gate_mid, down_mid;  // 128 x 128 tiles (before those below; down_split parts)
  int gate_skinny, down_skinny;   // few rows: the kernel made for them
  int gate_fused;          // 1: one kernel forms both products and the gated activation (no M x H round trip)
  int gate_pad, down_pad;  // the same kernels on zero-padded copies of the weights (widths off their tiles)
  int down_fast, up_wb, down_wb;
  int64_t ldg;             // pitch of G
  int g_blocked;           // the gated activation passes from the fused kernel to the down projection in 32 x 32 blocks, and the
                           // down projection reads its weights from a copy in such blocks
  F64Split up_s64, down_s64;   // fp32 storage
  int down_split;              // bf16, tiled: parts of the down projection's reduction
  size_t off_g, off_u, off_xtail, off_wt, off_wgp, off_wup, off_wdp, off_part, bytes;
};
bool make_ffn_plan(int dt, int64_t M, int64_t D, int64_t H, Room room, FfnPlan* q) {
  const bool split = room == Room::kAll || room == Room::kTight;
  if (dt != kF32 && dt != kBF16) return false;
  if (M < 0 || D < 1 || H < 1 || M > kMaxDim || D > kMaxDim || H > kMaxDim) return false;
  if (M * H > kMaxElems || M * D > kMaxElems || H * D > kMaxElems) return false;
  const size_t ts = dt == kF32 ? 4 : 2;
  const int64_t Mp = M > 0 ? M : 1;
  if (room == Room::kNoCopies && dt == kBF16 && mid_supported(Mp, D, H)) {
    // room for the activation alone: both products in 128 x 128 tiles, which need no copies
    *q = FfnPlan{};
    q->gate_mid = q->down_mid = 1; q->ldg = H; q->down_split = 1;
    q->off_part = q->bytes = align256((size_t)((Mp + 255) / 256 * 256) * H * ts);
    return true;
  }
  // off the tiles: padded copies, where the padding is not most of the work nor the launches most of the time
  const int64_t Hp = fast_gate_pad_h(H), Dq = fast_gate_pad_d(D), Dp = fast_pad_dim(D);
  const bool can_pad = dt == kBF16 && M >= 128 && M * D * H >= kStageFromWork && Hp * Dp <= 6 * H * D && (Hp / 128) * ((M + 255) / 256) <= (1 << 30);
  const GatePlan g = dt == kBF16 ? pick_gate(Mp, D, H, can_pad) : GatePlan{Gate::kSeparate, Xwt::kGeneric, 0.0, 0.0};
  q->gate_skinny = g.gate == Gate::kSkinny;
  q->gate_fused = g.gate == Gate::kTiled;
  q->gate_pad = g.gate == Gate::kPadded;
  q->ldg = q->gate_pad ? Hp : H;
  q->down_skinny = g.down == Xwt::kSkinny;
  q->down_fast = g.down == Xwt::kTiled;
  q->down_pad = g.down == Xwt::kPadded;
  q->up_wb = generic_wb(Mp, H);
  q->down_wb = generic_wb(Mp, D);
  size_t off = 0;
  const size_t mh = align256((size_t)((Mp + 255) / 256 * 256) * q->ldg * ts);
  q->off_g = off; off += mh;
  q->off_u = off; off += q->gate_fused || q->gate_skinny || q->gate_pad ? 0 : mh;    // the fused kernels never materialise the up product
  const size_t xpad = fast_padded_stages_x(D) ? (size_t)fast_padded_rows(Mp) * Dq * 2 : fast_padded_tail_bytes(D);
  q->off_xtail = off; off += align256(q->gate_pad ? xpad : (q->gate_fused ? fast_f1_tail_bytes(M, D) : 0));
  q->off_wgp = off; off += align256(q->gate_pad ? (size_t)Hp * Dq * 2 : 0);
  q->off_wup = off; off += align256(q->gate_pad ? (size_t)Hp * Dq * 2 : 0);
  q->off_wdp = off; off += align256(q->down_pad ? (size_t)Dp * Hp * 2 : 0);
  q->down_split = split && (q->down_pad || q->down_fast) ? fast_xwt_split(M, q->down_pad ? Hp : H, D) : 1;
  if (dt == kF32) {
    q->up_s64 = split ? f64_plan(Mp, H, D) : f64_unsplit(Mp, H, D);
    q->down_s64 = split ? f64_plan(Mp, D, H) : f64_unsplit(Mp, D, H);
  }
  const size_t up64 = dt == kF32 ? f64_part_bytes(q->up_s64) : 0;
  const size_t down = dt == kF32 ? f64_part_bytes(q->down_s64) : fast_xwt_part_bytes(M, D, q->down_split);
  q->off_part = off; off += align256(up64 > down ? up64 : down);
  q->gate_mid = q->down_mid = 0;
  if (dt == kBF16 && mid_supported(Mp, D, H)) {
    // either product, or both, where that is estimated to be faster (a padded gate product and its down product go together)
    int parts = 1;
    const double md = mid_margin(Mp) * mid_xwt_cost(Mp, H, D, mid_room(room, down), &parts), mg = mid_margin(Mp) * mid_gate_cost(Mp, D, H);
    const bool both = q->gate_pad || q->down_pad;
    q->gate_mid = both ? mg + md < g.gate_cost + g.down_cost : mg < g.gate_cost;
    q->down_mid = both ? q->gate_mid : md < g.down_cost;
    if (q->gate_mid) { q->ldg = H; q->gate_pad = 0; }
    if (q->down_mid) { q->down_split = parts; q->down_pad = 0; }
    const size_t sums = q->down_mid ? fast_xwt_part_bytes(M, D, parts) : down;
    if (q->off_part + align256(sums) > off) off = q->off_part + align256(sums);
  }
  q->g_blocked = q->gate_fused && !q->gate_mid && q->down_fast && !q->down_mid && M >= kCopyFromRows && q->down_split == 1;
  q->off_wt = off; off += align256(q->g_blocked ? (size_t)D * H * 2 : 0);
  q->bytes = off;
  return true;
}
}  // namespace

extern "C" size_t fdl_llama_ffn_workspace_bytes(fdl_dtype dt, int64_t M, int64_t D, int64_t H) {
  FfnPlan q;
  if (!make_ffn_plan((int)dt, M, D, H, Room::kAll, &q)) return 0;
  return q.bytes;
}

extern "C" fdl_status fdl_llama_ffn_forward(fdl_dtype dt, int64_t M, int64_t D, int64_t H, const void* X, const void* Wg,
                                            const void* Wu, const void* Wd, void* Y, void* workspace,
                                            size_t workspace_bytes, void* hip_stream) {
  if (!X || !Wg || !Wu || !Wd || !Y) return FDL_ERR_NULL;
  if (dt != FDL_F32 && dt != FDL_BF16) return FDL_ERR_DTYPE;
  FfnPlan q;
  const fdl_status st = fit_plan(workspace, workspace_bytes, &q,
                                 [&](Room room, FfnPlan* p) { return make_ffn_plan((int)dt, M, D, H, room, p); });
  if (st != FDL_OK) return st;
  if (!aligned(X, 16) || !aligned(Wg, 16) || !aligned(Wu, 16) || !aligned(Wd, 16) || !aligned(Y, 16)) return FDL_ERR_ALIGN;
  if (M == 0) return FDL_OK;
  clear_stale_error();
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(workspace);
  void* G = ws + q.off_g;
  void* U = ws + q.off_u;
  if (q.gate_pad || q.down_pad) {
    const int64_t Hp = fast_gate_pad_h(H), Dq = fast_gate_pad_d(D);
    StageJobs j = {};
    if (q.gate_pad) {
      stage_gate_x(&j, X, M, D, ws + q.off_xtail);
      stage_matrix(&j, Wg, H, D, D, ws + q.off_wgp, Hp, Dq);
      stage_matrix(&j, Wu, H, D, D, ws + q.off_wup, Hp, Dq);
    }
    if (q.down_pad) stage_matrix(&j, Wd, D, H, H, ws + q.off_wdp, fast_pad_dim(D), Hp);
    launch_stage(j, s);
  }
  if (q.gate_mid) {
    launch_mid_gate(M, D, H, X, Wg, Wu, G, s);
  } else if (q.gate_skinny) {
    launch_skinny_gate(M, D, H, X, Wg, Wu, G, s);
  } else if (q.gate_pad) {
    launch_fast_gate_padded(M, D, H, X, ws + q.off_xtail, ws + q.off_wgp, ws + q.off_wup, G, s);
  } else if (q.gate_fused) {
    launch_fast_gate(M, D, H, X, Wg, Wu, G, q.g_blocked != 0, ws + q.off_xtail, s);
  } else {
    GemmDesc g = {X, Wg, M, H, D, D, D, true, true, q.up_wb};
    if (dt == FDL_F32) launch_f64(0, g, q.up_s64, nullptr, nullptr, G, ws + q.off_part, s);
    else launch_generic_xwt(0, g, nullptr, nullptr, G, H, s);
    g.B = Wu;
    if (dt == FDL_F32) launch_f64(0, g, q.up_s64, nullptr, nullptr, U, ws + q.off_part, s);
    else launch_generic_xwt(0, g, nullptr, nullptr, U, H, s);
  }
  if (!q.gate_mid && !q.gate_fused && !q.gate_skinny && !q.gate_pad) launch_silu_mul((int)dt, M * H, G, U, G, s);
  if (q.down_mid) {
    launch_mid_xwt(0, M, H, D, G, Wd, nullptr, nullptr, Y, D, q.down_split, ws + q.off_part, s);
  } else if (q.down_pad) {
    launch_fast_down_padded(M, D, q.ldg, G, ws + q.off_wdp, Y, q.down_split, ws + q.off_part, s);
  } else if (q.down_skinny) {
    launch_skinny_xwt(0, M, H, D, G, Wd, nullptr, nullptr, Y, D, s);
  } else if (q.g_blocked) {
    launch_fast_block(D, H, Wd, ws + q.off_wt, s);
    launch_fast_xwt_blocked(M, H, D, G, ws + q.off_wt, Y, s);
  } else if (q.down_fast) {
    launch_fast_xwt(0, M, H, D, G, /*x_padded=*/true, Wd, nullptr, nullptr, Y, false, nullptr, s, q.down_split, ws + q.off_part);
  } else {
    GemmDesc g = {G, Wd, M, D, H, H, H, true, true, q.down_wb};
    if (dt == FDL_F32) launch_f64(0, g, q.down_s64, nullptr, nullptr, Y, ws + q.off_part, s);
    else launch_generic_xwt(0, g, nullptr, nullptr, Y, D, s);
  }
  return launch_status();
}
