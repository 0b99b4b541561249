// Internal launchers of libslse's device kernels.  Every launcher enqueues on
// `stream` and checks the launch; shapes are validated by the caller.
#pragma once

#include <vector>

#include "common.hpp"

namespace slse {

// --------------------------------------------------------------------------
// Fused residual-gradient (one pass over X): per-block partial sums of
//   X[0:n]^T (Y - X beta)   and   ||Y - X beta||^2
// written to partial[block][0..d] (index d holds the residual norm), to be
// summed by the next kernel on the stream.
// --------------------------------------------------------------------------
struct ResidGradPlan {
  int blocks = 0;
  int lpr = 0;   // lanes per row
  int vec = 0;   // elements per vector load
  int nch = 0;   // vector chunks per lane
  int ldp = 0;   // leading dimension of partial rows (>= d + 1)
  bool full = false;  // d = nch * lpr * vec: every lane's chunks are whole vectors
};

// lpr_hint > 0 picks the lane-group width (else a default); grid_blocks is the
// target grid, capped by `capacity` (the rows allocated for block partials).
ResidGradPlan plan_resid_grad(int64_t n, int d, slse_dtype storage, const void* X, int64_t ldx,
                              int grid_blocks, int capacity, int lpr_hint = 0);

struct UpdateArgs;

struct ResidGradArgs {
  int64_t n = 0;
  int d = 0;
  const void* X = nullptr;
  int64_t ldx = 0;
  const void* Y = nullptr;  // may be null (Y = 0)
  int64_t incy = 1;
  slse_dtype storage = SLSE_F64;
  slse_dtype accum = SLSE_F64;
  const double* beta = nullptr;
  double* partial = nullptr;  // [blocks][ldp]
  int capacity_blocks = 0;    // rows allocated in `partial`
  const int* done = nullptr;  // optional early-exit flag
  // an update that the pass takes first (its beta_next is then the pass's beta; `beta`
  // and `done` are not read); its partial rows are others than `partial`
  const UpdateArgs* step = nullptr;
};

// whether a pass of this shape can take the update u first
bool resid_grad_takes_step(const ResidGradPlan& pl, const UpdateArgs& u);
void launch_resid_grad(const ResidGradPlan& pl, const ResidGradArgs& a, hipStream_t s);

// g = scale * sum_r part[r][0..d) and, if given, rnorm2 = scale * sum_r part[r][d].
void launch_sum_rows(const double* part, int rows, int ldp, int d, double scale, double* g,
                     double* rnorm2, hipStream_t s);

// --------------------------------------------------------------------------
// M-IHS update (eqs. (98)/(99)) with the preconditioner M = H_hat^{-1}:
//   g      = scale * sum_rows part (+ w)
//   p      = M g
//   beta'  = beta + mu p + eta (beta - beta_prev)
// surrogate ||R^{-T} g||^2 = g . p is reduced into sur_out[0] (if given);
// when tol2 > 0 the step that brings it to <= tol2 * sur_ref[0] raises
// `done`, and later steps are skipped.
// --------------------------------------------------------------------------
struct UpdateArgs {
  const double* part = nullptr;  // [rows][ldp]: a pass's partial rows, or their sum (rows = 1)
  int rows = 0;                  // 0: g = w
  int ldp = 0;
  int d = 0;
  double scale = 1.0;
  const double* w = nullptr;  // added to g (adjoint right-hand side), may be null
  int64_t incw = 1;           // stride of w (0: w[0] for every k)
  const double* M = nullptr;
  int64_t ldm = 0;
  const double* beta = nullptr;
  const double* beta_prev = nullptr;
  double* beta_next = nullptr;
  double mu = 1.0;
  double eta = 0.0;
  double* beta_out = nullptr;     // copy of beta_next (may be null)
  double* traj_row = nullptr;     // copy of beta_next (may be null)
  double* sur_partial = nullptr;  // [blocks] scratch
  int* sur_counter = nullptr;     // zero before first use; left zero
  double* sur_out = nullptr;      // surrogate of this step (may be null)
  const double* sur_ref = nullptr;
  double tol2 = 0.0;
  int* done = nullptr;            // early-exit flag (may be null)
  int* status = nullptr;          // set to 1 on a non-finite surrogate (may be null)
};

int update_blocks(int d);
// whether the update of d columns sums a pass's partial rows itself (else it takes the
// sum of launch_sum_rows)
bool update_sums_rows(int d, int rows);
void launch_update(const UpdateArgs& a, hipStream_t s);

// rel_out[0] = ||beta - ref|| / ||ref|| and delta = beta - ref (either may be null).
void launch_iter_error(const double* beta, const double* ref, int d, double* rel_out,
                       double* delta, hipStream_t s);
// b0 = beta_out = traj_row = beta0 (zeros if null), b1 = beta_prev (if given), the
// four flags cleared (beta_out, traj_row may be null; the caller's arrays may alias)
void launch_iter_start(int d, const double* beta0, const double* beta_prev, double* b0, double* b1,
                       double* beta_out, double* traj_row, int* flags, hipStream_t s);
// out[0..3] = flags, out[4..6] = info, out[8..] = the T estimates (flags or sur may be
// null), written to pinned host memory
void launch_read_back(const int* flags, const int* info, const double* sur, int T, double* out,
                      hipStream_t s);
void launch_copy_f64(const double* src, double* dst, int64_t n, hipStream_t s);
void launch_fill_i32(int* dst, int value, int64_t n, hipStream_t s);
void launch_fill_f64(double* dst, double value, int64_t n, hipStream_t s);

// --------------------------------------------------------------------------
// SRHT: index maps and Walsh-Hadamard passes.
// --------------------------------------------------------------------------
struct SrhtArgs {
  slse_dtype t = SLSE_F64;
  int64_t N = 0;
  int d = 0;
  const void* X = nullptr;
  int64_t ldx = 0;
  const void* Y = nullptr;
  uint64_t seed = 0;
  int p = 0;  // N' = 2^p
  int64_t mK = 0;
  int64_t r = 0;
  void* A = nullptr;
  int64_t lda = 0;
  void* Ahat = nullptr;
  int64_t ldah = 0;
  // scratch
  int32_t* pi_sgn = nullptr;  // [N']
  int32_t* slotA = nullptr;   // [N']
  int32_t* slotH = nullptr;   // [N']
  void* Z = nullptr;          // [N'][ldz]
  int64_t ldz = 0;
  int ct = 0;                 // column tile (chosen by srht_plan)
  int bmax = 0;               // stages per pass cap
  bool xcd_swizzle = true;    // contiguous work runs per XCD
  bool indices_ready = false; // pi_sgn / slotA / slotH already built (batched)
  bool split_y = false;       // Y transformed on its own: Z = X's d columns, then N' values of Y
  bool y_pregathered = false; // (set at launch) Y gathered through P by the index-map kernel
};

void srht_plan(SrhtArgs& a, int prefer_ct);
// Single transforms whose X columns fill whole column tiles (d a multiple of
// the tile) take Y through its own one-column passes instead of a tile that
// would hold Y and padding (no-op otherwise; SLSE_SRHT_SPLIT_Y=0 disables).
void srht_split_y(SrhtArgs& a);

// Index maps of many SRHTs in one launch.  base/hbase: first global index of the
// job; rows, sign_words: the share of a block.
struct SrhtIndexJob {
  int64_t npad;
  int64_t r;
  int64_t mK;
  uint64_t seed;
  int p;
  int s0_last;
  int b_last;
  int rows;
  int sign_words;
  int pad_;
  int64_t base;
  int64_t hbase;
  int32_t* pi_sgn;
  int32_t* slotA;
  int32_t* slotH;
};

// p, npad and a block's share of a job
void srht_index_job(SrhtIndexJob& j, int p);
void srht_last_pass(const SrhtArgs& a, int* s0_last, int* b_last);
// index maps of B jobs (the same jobs on the device and on the host)
void launch_srht_index_batched(const SrhtIndexJob* jobs, const SrhtIndexJob* host_jobs, int B,
                               hipStream_t s);
size_t srht_z_bytes(const SrhtArgs& a);
void launch_srht(const SrhtArgs& a, hipStream_t s);

// SRHT passes of many transforms in shared launches (index maps already
// built, one workspace Z per multi-pass transform).  srht_batch_plan writes
// the device parameter records into `records` (host bytes, to be uploaded by
// the caller) and returns the launches; launch_srht_batched enqueues them.
struct SrhtBatchLaunch {
  int b = 0;     // butterfly stages of the pass
  int mode = 0;  // first / last pass flags
  int first = 0;  // first record of the launch
  int count = 0;  // transforms in the launch
  int64_t max_blocks = 0;
};
std::vector<SrhtBatchLaunch> srht_batch_plan(const std::vector<SrhtArgs>& as, slse_dtype t,
                                             std::vector<char>& records);
void launch_srht_batched(const std::vector<SrhtBatchLaunch>& L, const void* d_records, slse_dtype t,
                         hipStream_t s);
// --------------------------------------------------------------------------
// CountSketch and Gaussian sketches.
// --------------------------------------------------------------------------
struct CountSketchArgs {
  slse_dtype t = SLSE_F64;
  int64_t N = 0;
  int d = 0;
  const void* X = nullptr;
  int64_t ldx = 0;
  const void* Y = nullptr;
  uint64_t seed = 0;
  const int64_t* m = nullptr;
  int K = 0;
  int64_t r = 0;
  void* A = nullptr;  // levels back to back, m_1 first
  int64_t lda = 0;
  void* Ahat = nullptr;
  int64_t ldah = 0;
  void* scratch = nullptr;  // countsketch_scratch_bytes(*this) bytes: the bucket lists
};
size_t countsketch_scratch_bytes(const CountSketchArgs& a);
void launch_countsketch(const CountSketchArgs& a, hipStream_t s);

struct GaussianArgs {
  slse_dtype t = SLSE_F64;
  int64_t N = 0;
  int d = 0;
  const void* X = nullptr;
  int64_t ldx = 0;
  const void* Y = nullptr;
  uint64_t seed = 0;
  int64_t m = 0;
  uint64_t stream_id = 7;
  void* A = nullptr;
  int64_t lda = 0;
  float* partial = nullptr;   // split-K scratch
  double* partial64 = nullptr;
  int splits = 0;             // contiguous ranges of data rows, added in order
  int sub = 1;                // FP32 / FP64: parts that each range is summed in, in order too
  bool bf16 = false;          // BF16 operands on the matrix cores, FP32 accumulation
  bool tiles_ready = false;   // BF16: the scratch already holds this [X|Y]'s staged tiles
};
size_t gaussian_scratch_bytes(const GaussianArgs& a);
void gaussian_plan(GaussianArgs& a);
void launch_gaussian(const GaussianArgs& a, hipStream_t s);
void launch_debug_gaussian(uint64_t seed, uint64_t stream_id, int64_t k0, int64_t nk, int64_t j0,
                           int64_t nj, int form, double* out, hipStream_t s);
// the matrix-core form's generation of m x N entries of G alone (one checksum
// word per thread of `blocks` x 256 into sink)
void launch_gauss_generate(uint64_t seed, uint64_t stream_id, int64_t m, int64_t N, int blocks,
                           unsigned* sink, hipStream_t s);

// --------------------------------------------------------------------------
// Dense FP64 helpers for the factorization.
// --------------------------------------------------------------------------
// G = alpha A^T A (both triangles, ld ldg) for A rows x d in F32 or F64, summed in
// FP64.  Long A are split over rows into `scratch` (gram_scratch_doubles
// entries) and summed in split order.
// (FP64: A's entries are first scaled by a power of 2 near sqrt(alpha), so that only
// squares that alpha A^T A itself cannot hold leave the range; exact otherwise)
size_t gram_scratch_doubles(int64_t rows, int64_t d);
// scale = pre^2 rest, pre a power of 2 and rest in [1, 4) (FP32 data, whose squares FP64
// holds: pre = 1)
void gram_scale(double scale, slse_dtype at, double* pre, double* rest);
void launch_gram(int64_t rows, int d, double alpha, const void* A, int64_t lda, slse_dtype at,
                 double* G, int64_t ldg, double* scratch, size_t scratch_doubles, hipStream_t s);
// Q = alpha A Z^T (rows x d, ld d): A R^{-1} for Z = R^{-T}
void launch_times_inverse(int64_t rows, int d, double alpha, const void* A, int64_t lda,
                          slse_dtype at, const double* Z, double* Q, hipStream_t s);
// C0 = A0 B0 and C1 = A1 B1 (d x d, ld d; C with its own ld) in one launch
void launch_two_products(int d, const double* A0, const double* B0, double* C0, int64_t ldc0,
                         const double* A1, const double* B1, double* C1, int64_t ldc1,
                         hipStream_t s);
// R = upper Cholesky factor of the SPD d x d matrix G (R^T R = G, strict lower
// zeroed; R may be null) and Z = R^{-T} (d x d, ld d, strict upper zeroed).  G
// (ld d) is destroyed.  info[0] (zero on entry) becomes j + 1 of the first
// non-positive or non-finite pivot.
void launch_cholesky(int d, double* G, double* R, int64_t ldr, double* Z, int* info,
                     hipStream_t s);
// G += coef * trace(G) * I (d x d, ld = d).
void launch_shift_diag(int d, double* G, double coef, hipStream_t s);

// One Cholesky-route factorization of a batch: G = scale (pre A)^T (pre A), Z = R^{-T} of its
// Cholesky factor R, M = Z^T Z = G^{-1} (info[0]: first bad pivot + 1).  Every
// buffer is the job's own, row-major with leading dimension d (A: lda); G is
// destroyed and may be M.
struct FactorJob {
  const void* A = nullptr;
  int64_t lda = 0;
  int64_t rows = 0;
  int d = 0;
  double pre = 1.0, scale = 1.0;
  double* G = nullptr;
  double* Z = nullptr;
  double* M = nullptr;
  double* part = nullptr;  // splits x d x d partial Grams (factor_batched_splits > 1)
  int* info = nullptr;
};
// row splits of the batched Gram for sketches of at most rows_max rows
int factor_batched_splits(int64_t rows_max);
// All jobs at once (jobs in device memory; dmax, rows_max bound every job).
void launch_factor_batched(const FactorJob* jobs, int B, int dmax, int64_t rows_max,
                           slse_dtype at, hipStream_t s);

// --------------------------------------------------------------------------
// Adjoint rank-2 pass: dY = X lambda, dX = r lambda^T - (X lambda) beta^T.
// --------------------------------------------------------------------------
struct AdjointArgs {
  int64_t n = 0;
  int d = 0;
  const void* X = nullptr;
  int64_t ldx = 0;
  const void* Y = nullptr;
  slse_dtype t = SLSE_F64;
  const double* beta = nullptr;
  const double* lambda = nullptr;
  void* dX = nullptr;
  int64_t lddx = 0;
  void* dY = nullptr;
  slse_dtype gt = SLSE_F64;
};
void launch_adjoint(const AdjointArgs& a, hipStream_t s);

// --------------------------------------------------------------------------
// Batched M-IHS steps (many problems per launch).
// --------------------------------------------------------------------------
// batched residual-gradient pass: threads per block, and 16-byte vectors of
// [X|Y] a lane has in flight (a lane group's rows per step of its main loop
// are kBatchSlots / ch)
constexpr int kBatchThreads = 256;
constexpr int kBatchSlots = 8;
struct BatchStep {  // one problem at one global step
  const void* X;
  int64_t ldx;
  const void* Y;
  int64_t incy;
  int64_t n;  // rows of this step (0: the problem is idle)
  double scale;
  const double* beta;
  const double* beta_prev;
  double* beta_next;
  int ntiles;
  int tile_rows;  // rows per tile in this step (the last tile may be short)
};
struct BatchProblem {
  int d;
  int lpr;  // lanes per row (a power of 2 <= 64)
  int ch;   // 16-byte vectors per lane per row (1, 2 or 4)
  int64_t part_off;  // first partial row of this problem in the pool
  const double* M;
  double* beta_out;
  double mu, eta;
  const double* beta0;  // initial iterate (device) or null for 0
  double* beta_init;    // the iterate buffer the first step reads
};
void launch_batched_resid_grad(const BatchStep* steps, const BatchProblem* probs, const int* prefix,
                               int B, int total_tiles, int grid, double* pool, slse_dtype t, bool vec,
                               int chmax, hipStream_t s);
void launch_batched_update(const BatchStep* steps, const BatchProblem* probs, int B, int dmax,
                           const double* pool, int* flags, hipStream_t s);
// beta_init = beta_out = beta0 (or 0) for every problem
void launch_batched_init(const BatchProblem* probs, int B, int dmax, hipStream_t s);

// --------------------------------------------------------------------------
// Test hooks.
// --------------------------------------------------------------------------
// Reference streams (no method arithmetic): mode 0 reads `bytes` of src (one
// word per block into dst[0..blocks)), mode 1 copies src to dst.
void launch_stream_reference(int mode, const void* src, void* dst, int64_t bytes, int blocks,
                             hipStream_t s);
void launch_debug_stream(int what, uint64_t seed, int stream_id, int64_t aux, int64_t start,
                         int64_t count, int64_t* out, hipStream_t s);

}  // namespace slse
