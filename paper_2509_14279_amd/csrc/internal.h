// Host-side declarations shared by the translation units of libfdl: the launch plan (which
// kernels run, how the workspace is carved up) and one launcher per phase of the block.
//
// Phases:  F1  Zsave = X W^T + b
//          F2  mean, rstd of GELU(Zsave), Y = (GELU(Zsave) - mean) rstd gamma + beta   (one kernel)
//          B1  dZ and the column partials of dbeta, dgamma, db  (B1a: row sums c1, c2 first)
//          B2  column partials -> dbeta, dgamma, db
//          B3  dX = dZ W            B4  dW = dZ^T X
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace fdl {

enum DType { kF32 = 0, kBF16 = 1 };

// How a product in fp64 is dealt out (gemm_f64.hip): tiles done as a whole, tiles split into `split` parts
// (small: in 32 x 32 tiles, none split; the rest, and the room, are what would be otherwise)
struct F64Split { int64_t whole, parted; int split, small; };

// The two contractions that end a backward pass: dX [M,K] = dZ W, dW [N,K] = dZ^T X.
struct GradPlan {
  int dt;
  int64_t M, K, N;
  int b3_fast, b4_fast;   // dX, dW on the tuned kernels
  int b3_wb, b4_wb;
  int pad;                // 1: padded mode of the fast contractions (N, K not both multiples of 256)
  int stage_x;            // 1 (padded mode): X goes through a copy with pitch Kp
  int64_t ldz;            // pitch of the dZ buffer in elements (N, or N rounded up to 256 in padded mode)
  int blocked;            // 1: dZ lives in 32 x 32 blocks (its writer -> tuned dX and dW kernels only)
  int64_t b4_fast_rows;   // rows of dW's reduction the fast kernel covers
  int extra;              // 1: the generic kernel adds a partial sum for the rows after them
  int pair;               // 1: both contractions share one launch
  int split_a, split_b;   // parts of the reductions over N (dX) and over M (dW)
  int parts_b;            // partial sums of dW: split_b + extra
  size_t off_dz;          // T [M rounded up to 256][ldz]
  size_t off_dxpart;      // float [split_a][M][K]   (split_a > 1)
  size_t off_dwpart;      // float [parts_b][N][K]   (parts_b > 1)
  size_t off_wpad, off_xpad;   // zero-padded copies of W and (stage_x) X
  int mid;                // 1: both contractions in 128 x 128 tiles, in one launch (gemm_mid.hip); the fields above say what would
                          //    run otherwise, pitch and parts are this path's
  F64Split s64_a, s64_b;  // fp32 storage: dX, dW
  size_t off_part64_a, off_part64_b;   // their split tiles' sums
};

struct Plan {
  int dt;
  int64_t M, K, N;
  // forward
  int f1_mid;             // 1: 128 x 128 tiles (before those below); f1_split parts, their sums at off_part
  int f1_skinny;          // 1: bf16 kernel for few rows (before the two below)
  int f1_fast;            // 1: bf16 fast MFMA kernel, 0: generic kernel
  int f1_wb;              // generic kernel: 16x16 blocks per wave tile side (wave tile = 16*wb)
  size_t off_rows;        // F2's scratch for rows beyond its registers, the first
  F64Split f1_s64;        // fp32 storage
  int f1_split;           // bf16, tiled: parts of the reduction where there are few tiles
  size_t off_part;        // their sums
  size_t fwd_bytes;
  size_t static_need;     // what fdl_forward_static compares with its array (the header's rule)
  // backward
  int b1_fused;           // 1: one pass with the row held in registers; 0: B1a + B1b
  int b1_groups;          // number of row groups that produce column partials
  int b1_rows_per_group;  // B1b only
  GradPlan g;             // dX and dW
  int pad;                // forward: padded mode of the fast contraction (N, K not both multiples of 256)
  int stage_x;            // forward, padded mode: X goes through a copy with pitch Kp
  size_t off_wpad_f, off_bpad_f;   // forward: zero-padded copies of W [Np][Kp] and b [Np]
  size_t off_xtail;       // forward: padded copy of X's last rows (ragged M on the fast path), or of X
  size_t off_c12;         // C [2][M]
  size_t off_colpart;     // C [groups][3][N]
  size_t bwd_bytes;
  size_t bytes;           // max(fwd, bwd)
};

// What a plan may use the workspace for: everything; for the sums of split reductions in 128 x 128 tiles only what the other
// kernels would use; no partial sums of split reductions; nor, in the forward products, copies of the operands (the kernels that
// need none then form them).
enum class Room { kAll, kTight, kNoSplit, kNoCopies };
void make_grad_plan(int dt, int64_t M, int64_t K, int64_t N, Room room, bool may_block, size_t* off, GradPlan* p);
// Returns false when the shape or dtype is not supported.  forward_only: the backward pass is not planned (bytes stays 0).
bool make_plan(int dt, int64_t M, int64_t K, int64_t N, Room room, Plan* p, bool forward_only = false);

// ---- per-device facts and per-call failure notes --------------------------------------------------
// Compute units and accelerator dies (each die has its own L2) of the calling thread's current device, queried from
// the runtime once per device.  Returns false (and leaves a note, see below) if the query fails.
struct DeviceInfo { int cus; int xcds; };
bool device_info(DeviceInfo* out);

// A launcher that cannot launch (a failed attribute call, a failed device query) prints the reason to stderr and
// leaves a note for the calling thread; the entry point turns a note into FDL_ERR_LAUNCH.
void note_failure(const char* what, hipError_t e);

// Raise the dynamic-LDS limit of a kernel once per device (flags: one byte per device ordinal, zero-initialised,
// owned by the caller - one array per kernel instantiation).  Safe to call from several host threads.
constexpr int kMaxDevices = 64;
struct OnceFlags { std::atomic<unsigned char> done[kMaxDevices]; };
bool ensure_dynamic_lds(const void* kernel, int bytes, OnceFlags* flags);

// ---- generic bf16 MFMA GEMM: C[i][j] = sum_r A(i,r) B(j,r), any shape, any alignment ------------
// a_rc / b_rc: the operand is contiguous along the reduction index r (element (i,r) at A[i*ld + r]);
// otherwise it is contiguous along i (element (i,r) at A[r*ld + i]).
struct GemmDesc {
  const void* A; const void* B;
  int64_t I, J, R;
  int64_t lda, ldb;
  bool a_rc, b_rc;
  int wb;
};
int generic_wb(int64_t I, int64_t J);        // GemmDesc::wb
// forward-product orientation with an optional bias and a ReLU or ReLU-mask epilogue (sibling operators)
void launch_generic_xwt(int kind, const GemmDesc& g, const float* bias, const void* aux, void* C, int64_t ldc, hipStream_t s);
double generic_xwt_cost(int64_t M, int64_t K, int64_t N);
// plain store: C [I][J]
void launch_generic_store(const GemmDesc& g, void* C, hipStream_t s);
// plain store of the fp32 accumulators: C [I][J] float (bf16 storage; a partial sum for launch_finish)
void launch_generic_store_f32(const GemmDesc& g, float* C, hipStream_t s);

// ---- fp32-storage contractions in fp64 (gemm_f64.hip): GemmDesc as above, any shape ---------------
F64Split f64_plan(int64_t I, int64_t J, int64_t R);
// dx, dw: what would run otherwise, or null: no room for its sums
bool f64_small_grads(int64_t M, int64_t K, int64_t N, const F64Split* dx, const F64Split* dw);
size_t f64_part_bytes(const F64Split& q);
void launch_f64(int kind, const GemmDesc& g, const F64Split& q, const float* bias, const void* aux, void* C, void* part,
                hipStream_t s);

// the parts of a product whose tiles are all split (q.whole = 0), left for launch_f2_sums: Z [I][J] = their sums + bias
struct F64Sums { const double* part; const float* bias; float* Z; int64_t stride; int split, tiles_j; };
F64Sums launch_f64_parts(const GemmDesc& g, const F64Split& q, const float* bias, void* Z, void* part, hipStream_t s);

// ---- row-wise / column-wise phases ------------------------------------------------------------
// row statistics of GELU(Zsave) and the normalised output (Zsave and Y may be the same buffer); part: f2_part_bytes of scratch
size_t f2_part_bytes(int dt, int64_t M, int64_t N);
void launch_f2(int dt, int64_t M, int64_t N, float eps, const void* Zsave, const float* gamma, const float* beta, void* Y,
               float* mean, float* rstd, void* part, hipStream_t s);
bool f2_takes_sums(int64_t N);
void launch_f2_sums(int64_t M, int64_t N, float eps, const F64Sums& q, const float* gamma, const float* beta, void* Y, float* mean,
                    float* rstd, hipStream_t s);
void launch_b1a(int dt, int64_t M, int64_t N, const void* dY, const void* Zsave, const float* gamma,
                const float* mean, const float* rstd, void* c12, hipStream_t s);
// ldz: pitch of dZ in elements (N, or N rounded up to the tile in the padded mode of the fast contractions)
void launch_b1b(int dt, int64_t M, int64_t N, int64_t ldz, int rows_per_group, int groups, const void* dY, const void* Zsave,
                const float* gamma, const float* mean, const float* rstd, const void* c12, void* dZ,
                void* colpart, hipStream_t s);
// fused single pass (row held in registers; ldz: pitch of dZ, whose surplus columns it zeroes); returns false if the row
// is too long for it
bool b1_fused_supported(int dt, int64_t N, int64_t ldz);
int b1_fused_groups(int dt, int64_t M, int64_t N);   // number of row groups it should be launched with (before capping at M)
int b1_fused_slots(int dt, int64_t N, int64_t ldz);   // rows that a group has in hand at once
int b1b_rows_per_group(int dt, int64_t M, int64_t N);
void launch_zero_cols_bf16(void* dZ, int64_t M, int64_t N, int64_t ldz, hipStream_t s);
// blocked: dZ is written as [M / 32][N / 32] blocks of 32 x 32 elements (bf16, M and N multiples of 32, ldz = N)
void launch_b1_fused(int dt, int64_t M, int64_t N, int64_t ldz, int groups, bool blocked, const void* dY, const void* Zsave,
                     const float* gamma, const float* mean, const float* rstd, void* dZ, void* colpart, hipStream_t s);
// bf16 storage
void launch_b2(int64_t N, int groups, const void* colpart, float* dbeta, float* dgamma, float* db, hipStream_t s);
// bf16: the column sums (as launch_b2) and up to two sums of fp32 split-reduction partials
// (out[k][i] = bf16(sum over q < parts[k] of part[k][q * partial_stride(n[k]) + i]); parts[k] = 0: none) in one launch
struct TailSums {
  const float* part[2];
  int parts[2];
  int64_t n[2];
  void* out[2];
  int blocks[2];          // filled in by launch_finish, as stride
  int64_t stride[2];
  const float* colpart;
  int groups;
  int64_t N;
  int kinds;              // kinds of column sum: colpart [groups][kinds][N] -> col_out
  float* col_out[3];
};
void launch_finish(TailSums j, hipStream_t s);
// fp32 storage: both gradient contractions in one launch; then their split tiles' sums and the column sums (j.colpart holds
// doubles, j's split products unused) in another
struct F64Grads { GemmDesc dx, dw; F64Split qx, qw; void *dX, *partx, *dW, *partw; };
void launch_f64_grads(const F64Grads& a, const TailSums& j, hipStream_t s);
void launch_f64_grads_finish(const F64Grads& a, const TailSums& j, hipStream_t s);

// ---- sibling operators' row-wise / element-wise kernels ------------------------------------------
void launch_layernorm(int dt, int64_t M, int64_t N, float eps, const void* A, const float* gamma, const float* beta,
                      void* Y, float* mean, float* rstd, hipStream_t s);
void launch_rmsnorm(int dt, int64_t M, int64_t N, float eps, const void* A, const float* weight, void* Y, hipStream_t s);
int colsum_groups(int64_t M);
// ldg: pitch of G; blocked: G is stored in 32 x 32 blocks (bf16; M, N multiples of 32)
void launch_colsum_partial(int dt, int64_t M, int64_t N, int64_t ldg, const void* G, bool blocked, void* colpart, hipStream_t s);
void launch_colsum_finish(int64_t M, int64_t N, const void* colpart, float* out, hipStream_t s);
void launch_silu_mul(int dt, int64_t n, const void* G, const void* U, void* H, hipStream_t s);

// ---- bf16 products with few rows (gemm_skinny.hip): any K and N -----------------------------------
// Which kernel forms the forward product [M,K] x [N,K]^T (see gemm_skinny.hip)
enum class Xwt { kGeneric, kSkinny, kTiled, kPadded };
// may_copy: into padded or partly copied operands; may_pad: into padded ones; x_padded: X has readable rows behind a partial tile
Xwt pick_xwt(int64_t M, int64_t K, int64_t N, bool may_copy = true, bool may_pad = true, bool x_padded = false, double* cost = nullptr);
// and the gate and up products of the feed-forward block, [M,D] x [H,D]^T twice, then its down product
enum class Gate { kSeparate, kSkinny, kTiled, kPadded };
struct GatePlan { Gate gate; Xwt down; double gate_cost, down_cost; };
GatePlan pick_gate(int64_t M, int64_t D, int64_t H, bool can_pad);
void launch_skinny_xwt(int kind, int64_t M, int64_t K, int64_t N, const void* X, const void* W, const float* bias,
                       const void* aux, void* out, int64_t ldo, hipStream_t s);
void launch_skinny_gate(int64_t M, int64_t D, int64_t H, const void* X, const void* Wg, const void* Wu, void* out, hipStream_t s);

// ---- bf16 fast path -----------------------------------------------------------------------------
// F1 and B3 accept any M >= 128 (the last row tile may be partial); N, K as the tiles and the pipeline require.
bool fast_f1_supported(int64_t M, int64_t K, int64_t N);
bool fast_b3_supported(int64_t M, int64_t K, int64_t N);
// B4 reduces over M: the fast kernel takes the first fast_b4_rows(M) rows; the rest (< 128) is left to the caller
bool fast_b4_supported(int64_t M, int64_t K, int64_t N);
int64_t fast_b4_rows(int64_t M);
size_t fast_f1_tail_bytes(int64_t M, int64_t K);
// Wb [N][K]: W in blocks of 32 x 32 (N, K multiples of 64)
void launch_fast_block(int64_t N, int64_t K, const void* W, void* Wb, hipStream_t s);
// zero-padded copies of up to four matrices and one vector in one launch (see stage_kernel)
struct StageJob { const void* src; void* dst; int64_t rows, cols, ld, rows_out, cols_out; int blocks; };
struct StageJobs { StageJob job[4]; int count; const float* vsrc; float* vdst; int64_t vn, vn_out; };
void stage_matrix(StageJobs* j, const void* src, int64_t rows, int64_t cols, int64_t ld, void* dst, int64_t rows_out, int64_t cols_out);
void stage_vector(StageJobs* j, const float* src, int64_t n, float* dst, int64_t n_out);
void launch_stage(const StageJobs& j, hipStream_t s);
// padded mode (N, K not both multiples of 256): see gemm_bf16.hip
constexpr int64_t kStageFromWork = (int64_t)1 << 28;   // M N K from which odd rows are worth copying
bool fast_padded_supported(int64_t M, int64_t K, int64_t N);
bool fast_padded_stages_x(int64_t K);          // X goes through a copy with pitch Kp (else only its last row tile is copied)
bool fast_padded_can_skip_copy(int64_t K);
int64_t fast_pad_dim(int64_t n);
int64_t fast_padded_rows(int64_t M);           // rows of that copy, and of dZ
size_t fast_padded_tail_bytes(int64_t K);
inline size_t fast_padded_x_bytes(int64_t M, int64_t K, bool staged) {
  return staged ? (size_t)fast_padded_rows(M) * fast_pad_dim(K) * 2 : fast_padded_tail_bytes(K);
}
int64_t fast_padded_b4_rows(int64_t M, int64_t K);
void stage_padded(StageJobs* j, int64_t M, int64_t K, int64_t N, bool staged, const void* X, const void* W, const float* bias,
                  void* xw, void* Wp, float* biasp);
void launch_fast_xwt_padded(int kind, int64_t M, int64_t K, int64_t N, bool staged, const void* X, const void* xw, const void* Wp,
                            const float* biasp, const void* aux, void* out, int split, void* part, hipStream_t s);
// parts of the forward product's reduction where it has few tiles, and their fp32 sums
int fast_xwt_split(int64_t M, int64_t K, int64_t N);
double fast_xwt_cost(int64_t M, int64_t K, int64_t N, int* split);    // estimated time, us
size_t fast_xwt_part_bytes(int64_t M, int64_t N, int split);
int64_t fast_gate_pad_h(int64_t H);
int64_t fast_gate_pad_d(int64_t D);
void stage_gate_x(StageJobs* j, const void* X, int64_t M, int64_t D, void* xw);
void launch_fast_gate_padded(int64_t M, int64_t D, int64_t H, const void* X, const void* xw, const void* Wgp, const void* Wup,
                             void* Hout, hipStream_t s);
void launch_fast_down_padded(int64_t M, int64_t D, int64_t Hp, const void* G, const void* Wdp, void* out, int split, void* part,
                             hipStream_t s);
// fp32 partial sums of n elements lie this far apart (16-byte parts)
inline int64_t partial_stride(int64_t n) { return (n + 3) & ~(int64_t)3; }
void launch_fast_b3_padded(int64_t M, int64_t K, int64_t N, const void* dZ, const void* Wp, void* dX, hipStream_t s);
void launch_fast_b4_padded(int64_t M, int64_t K, int64_t N, int split, int extra, const void* dZ, const void* X, int64_t ldx,
                           void* dW, void* dwpart, hipStream_t s);
// the forward product, also of the sibling operators (see gemm_bf16.hip); shapes as fast_f1_supported
void launch_fast_xwt(int kind, int64_t M, int64_t K, int64_t N, const void* X, bool x_padded, const void* W,
                     const float* bias, const void* aux, void* out, bool out_blocked, void* xtail,
                     hipStream_t s, int split = 1, void* part = nullptr);     // see fast_xwt_split
// the plain product of an X in 32 x 32 blocks (rows padded to whole tiles) and weights from launch_fast_block
constexpr int64_t kCopyFromRows = 16384;   // batch size from which the feed-forward block's down product runs so
void launch_fast_xwt_blocked(int64_t M, int64_t K, int64_t N, const void* X, const void* Wb, void* out, hipStream_t s);
// gate and up products of the feed-forward block with the gated activation in the epilogue (see gemm_bf16.hip)
bool fast_gate_supported(int64_t M, int64_t D, int64_t H);
void launch_fast_gate(int64_t M, int64_t D, int64_t H, const void* X, const void* Wg, const void* Wu, void* Hout, bool out_blocked,
                      void* xtail, hipStream_t s);
// dZ must have readable rows up to the next multiple of 256
// dz_blocked: dZ is stored in 32 x 32 blocks (launch_b1_fused with blocked = true; M, N multiples of 32)
void launch_fast_b3(int64_t M, int64_t K, int64_t N, const void* dZ, bool dz_blocked, const void* W, void* dX,
                    hipStream_t s);
int fast_b4_split(int64_t M, int64_t K, int64_t N);
void launch_fast_b4(int64_t M, int64_t K, int64_t N, int split, int extra, const void* dZ, bool dz_blocked, const void* X,
                    void* dW, void* dwpart, hipStream_t s);
// dX and dW in one launch where together they have at most a tile per compute unit; sa, sb: parts of the two reductions
bool fast_pair_plan(int64_t M, int64_t K, int64_t N, int64_t rows, int* sa, int* sb);
struct PairArgs {
  int64_t M, K, N, rows;       // rows: of the dW reduction
  int sa, sb, extra;
  const void* dZ; int64_t ldz; bool dz_blocked;
  const void* W; int64_t ldw;
  const void* X; int64_t ldx;
  void* dX; void* dxpart; void* dW; void* dwpart;
};
void launch_fast_pair(const PairArgs& a, hipStream_t s);
// out = f(the parts' sums + bias), kinds as launch_fast_xwt; parts [M][N] fp32, stride elements apart
void launch_xwt_reduce(int kind, int split, const void* part, int64_t stride, int64_t M, int64_t N, const float* bias, const void* aux,
                       void* out, int64_t ldo, hipStream_t s);

// ---- bf16 products in 128 x 128 tiles (gemm_mid.hip): any alignment, no copies; K, N >= 8 ---------
bool mid_supported(int64_t M, int64_t K, int64_t N);
// estimated times, us, and the parts of the reductions that give them; room: bytes for the parts' fp32 sums
double mid_xwt_cost(int64_t M, int64_t K, int64_t N, size_t room, int* split);
double mid_margin(int64_t M);
double mid_grads_cost(int64_t M, int64_t K, int64_t N, size_t room, int* sa, int* sb);
// as launch_fast_xwt (kind 2 leaves columns of out behind N as they are); part: fast_xwt_part_bytes(M, N, split)
void launch_mid_xwt(int kind, int64_t M, int64_t K, int64_t N, const void* X, const void* W, const float* bias, const void* aux,
                    void* out, int64_t ldo, int split, void* part, hipStream_t s);
// gate and up products of the feed-forward block with the gated activation
double mid_gate_cost(int64_t M, int64_t D, int64_t H);
void launch_mid_gate(int64_t M, int64_t D, int64_t H, const void* X, const void* Wg, const void* Wu, void* out, hipStream_t s);
// dX and dW in one launch; split reductions leave fp32 sums as launch_fast_pair, unsplit ones finish the column sums `cols` too
struct MidGrads {
  int64_t M, K, N;
  int sa, sb;
  const void* dZ; int64_t ldz;
  const void* W; const void* X;
  void* dX; void* dxpart; void* dW; void* dwpart;
  TailSums cols;
};
void launch_mid_grads(const MidGrads& a, hipStream_t s);

}  // namespace fdl
