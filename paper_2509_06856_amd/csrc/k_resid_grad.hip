// Fused residual-gradient pass g = X^T (Y - X beta) (the full-data gradient
// of eq. (99), and of eq. (98) on a sketched prefix), reading X once.
//
// Layout: a row of X is split over a group of `lpr` lanes; lane l of the group
// owns the vector chunks c*lpr + l (c < NCH) of VEC consecutive elements, so a
// wave's loads of one row are contiguous.  Rows may start at any element: the
// 16-byte loads need no 16-byte alignment, and where d is no multiple of the
// chunks the last one is moved back to end with the row, its elements that
// another lane owns replaced by zeros (1000003 x 101 float32: 377 us with
// element loads behind a guard each, 93 us so).  Per row the group forms the partial
// dot x_j . beta, all-reduces it across its lanes (xor shuffles), and every
// lane folds r_j = y_j - x_j . beta into its own slice of g.  A wave streams
// 64/lpr rows per step, UNROLL steps in flight, over one contiguous chunk of
// rows per block.  At the end the wave's row
// groups, then the block's waves, are summed; the block writes one partial
// row, and the kernel that follows on the stream (the sum below, or the update
// step of a narrow problem) adds the rows in a fixed order (deterministic for a
// fixed launch shape).  The kernel boundary is the hand-off: a ticket per
// block, with the release and acquire it needs across the XCDs' caches, cost
// about 50 ns a block one after another (1000003 x 101 float32: 93, 106 and 139 us
// on 256, 512 and 1024 blocks with tickets, 88, 88 and 88 without; 2^20 x 256:
// 170.9 -> 164.2 us; the mixed solve at 2^22 x 512 43.5 -> 42.2 ms).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "update_step.hpp"

namespace slse {
namespace {

// Build-time launch shape: threads per block and bytes in flight per lane (in
// units of 256 B) of the fully vectorised main loop.
#ifndef SLSE_RG_THREADS
#define SLSE_RG_THREADS 256
#endif
#ifndef SLSE_RG_DEPTH
#define SLSE_RG_DEPTH 1
#endif
constexpr int kThreads = SLSE_RG_THREADS;
constexpr int kWaves = kThreads / 64;

// a vector of VEC elements whose address is a multiple of the element size
template <typename T, int VEC>
struct VecT {
  typedef T type __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
};
template <typename T>
struct VecT<T, 1> {
  using type = T;
};

template <typename T, int VEC>
__device__ __forceinline__ void load_vec(const T* __restrict__ p, T (&v)[VEC]) {
  using V = typename VecT<T, VEC>::type;
  const V x = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  if constexpr (VEC == 1) {
    v[0] = x;
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = x[i];
  }
}

// x widened to the accumulation type
template <typename Acc, typename T>
__device__ __forceinline__ Acc widen(T x) {
  return (Acc)x;
}

// The same, as a separate instruction the compiler cannot merge with `widen`:
// the widened row is then not kept alive from the dot to the update.
template <typename Acc, typename T>
__device__ __forceinline__ Acc widen_again(T x) {
  if constexpr (sizeof(Acc) == 8 && sizeof(T) == 4) {
    double r;
    asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
  } else {
    return (Acc)x;
  }
}

// value of lane (lane ^ m) for 32- or 64-bit values (m < 64, no width clamp)
template <typename V>
__device__ __forceinline__ V lane_xor(V v, int m, int lane) {
  const int addr = (lane ^ m) << 2;
  if constexpr (sizeof(V) == 8) {
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)(u & 0xffffffffll));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(u >> 32));
    return __builtin_bit_cast(V, ((long long)hi << 32) | (unsigned int)lo);
  } else {
    return __builtin_bit_cast(V, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, v)));
  }
}

template <typename T, int VEC, int NCH, int DEPTH = 1>
constexpr int unroll_for() {
  constexpr int bytes = NCH * VEC * (int)sizeof(T);
  constexpr int u = 256 * DEPTH / bytes;
  return u < 1 ? 1 : (u > 16 * DEPTH ? 16 * DEPTH : u);
}

// FULL: d = NCH * lpr * VEC, so every chunk is a whole vector inside the row.
// Otherwise NCH is the exact chunk count (d > (NCH - 1) lpr VEC) and only the
// last chunk can reach past the row.
template <typename T, typename Acc, int VEC, int NCH, bool HAS_Y, bool FULL>
__device__ __forceinline__ void resid_grad(int64_t n, int d, const T* __restrict__ X, int64_t ldx,
                                           const T* __restrict__ Y, int64_t incy, const double* beta,
                                           int lpr, double* __restrict__ partial, int ldp) {
  constexpr int UNROLL = unroll_for<T, VEC, NCH, SLSE_RG_DEPTH>();
  __shared__ double s_red[kWaves][1025];

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int gpw = 64 / lpr;  // row groups per wave
  const int grp = lane / lpr;
  const int l = lane - grp * lpr;

  // the last chunk: its first column, and which of its elements this lane owns
  const int col_last = ((NCH - 1) * lpr + l) * VEC;
  const int off_last = FULL ? col_last : min(col_last, d - VEC);
  auto owns = [&](int c, int v) { return FULL || c < NCH - 1 || off_last + v >= col_last; };
  auto offset = [&](int c) { return c == NCH - 1 ? off_last : (c * lpr + l) * VEC; };

  // beta slice of this lane
  Acc b[NCH][VEC];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int v = 0; v < VEC; ++v) b[c][v] = owns(c, v) ? (Acc)beta[offset(c) + v] : (Acc)0;

  Acc acc[NCH][VEC];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[c][v] = 0;
  Acc rr = 0;

  // each block streams one contiguous chunk of rows; at every unroll step its
  // lane groups cover `rs` consecutive rows
  const int rs = kWaves * gpw;
  const int64_t chunk = round_up(ceil_div(n, (int64_t)gridDim.x), rs);
  const int64_t r0 = (int64_t)blockIdx.x * chunk;
  const int64_t r1 = min(n, r0 + chunk);

  // UNROLL rows per lane group, from `row0` every rs rows.  PART: some of them
  // may lie past r1; those read row r1 - 1 and count as zeros (their residuals too:
  // the dot of zeros with an infinite beta is NaN).
  auto step = [&](int64_t row0, auto part) {
    constexpr bool PART = decltype(part)::value;
    T x[UNROLL][NCH][VEC];
    T y[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      int64_t row = row0 + (int64_t)u * rs;
      if constexpr (PART) row = min(row, r1 - 1);
      const T* xr = X + row * ldx;
#pragma unroll
      for (int c = 0; c < NCH; ++c) load_vec<T, VEC>(xr + offset(c), x[u][c]);
      if constexpr (HAS_Y) {
        y[u] = __builtin_nontemporal_load(Y + row * incy);
      } else {
        y[u] = 0;
      }
    }
    if constexpr (!FULL) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
#pragma unroll
        for (int v = 0; v < VEC; ++v) x[u][NCH - 1][v] = owns(NCH - 1, v) ? x[u][NCH - 1][v] : (T)0;
    }
    if constexpr (PART) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const bool in = row0 + (int64_t)u * rs < r1;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
          for (int v = 0; v < VEC; ++v) x[u][c][v] = in ? x[u][c][v] : (T)0;
      }
    }
    // partial dots row by row (the widened values of a row die with its dot)
    Acc dot[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      __builtin_amdgcn_sched_barrier(0);
      Acc p0 = 0, p1 = 0;
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          if ((c * VEC + v) & 1)
            p1 = fma(widen<Acc>(x[u][c][v]), b[c][v], p1);
          else
            p0 = fma(widen<Acc>(x[u][c][v]), b[c][v], p0);
        }
      dot[u] = p0 + p1;
    }
    __builtin_amdgcn_sched_barrier(0);
    // all-reduce the rows' dots inside each lane group, the rows interleaved
    for (int m = lpr >> 1; m > 0; m >>= 1) {
      Acc o[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) o[u] = lane_xor(dot[u], m, lane);
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) dot[u] += o[u];
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      Acc r = (Acc)y[u] - dot[u];
      if constexpr (PART) r = row0 + (int64_t)u * rs < r1 ? r : (Acc)0;
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[c][v] = fma(r, widen_again<Acc>(x[u][c][v]), acc[c][v]);
      rr = fma(r, r, rr);
    }
  };
  // whole steps while every row of the step is in range for the whole wave
  // (the bound is wave-uniform: no guards and no branches), then one last step
  // that may reach past the chunk
  const int64_t last_off = (int64_t)(gpw - 1) + (int64_t)(UNROLL - 1) * rs;
  int64_t wb = r0 + wave * gpw;
  for (; wb + last_off < r1; wb += (int64_t)rs * UNROLL) step(wb + grp, std::false_type{});
  if (wb < r1) step(wb + grp, std::true_type{});

  // sum the wave's row groups: lanes with equal l hold the same columns
  double accd[NCH][VEC];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      double t = (double)acc[c][v];
      for (int m = lpr; m < 64; m <<= 1) t += wave_xor(t, m);
      accd[c][v] = t;
    }
  double rrd = (double)rr;  // every lane of a group holds the same r: count lane l == 0 only
  rrd = (l == 0) ? rrd : 0.0;
  for (int m = 1; m < 64; m <<= 1) rrd += wave_xor(rrd, m);

  // block reduction through LDS (columns d.. handled by the spill loop below)
  double* prow = partial + (int64_t)blockIdx.x * ldp;
  for (int c0 = 0; c0 < d + 1; c0 += 1024) {
    if (grp == 0) {
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          const int col = offset(c) + v;
          if (owns(c, v) && col >= c0 && col < c0 + 1024) s_red[wave][col - c0] = accd[c][v];
        }
      if (l == 0 && d >= c0 && d < c0 + 1024) s_red[wave][d - c0] = rrd;
    }
    __syncthreads();
    for (int col = c0 + threadIdx.x; col < min(d + 1, c0 + 1024); col += kThreads) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) t += s_red[w][col - c0];
      prow[col] = t;
    }
    __syncthreads();
  }
}

template <typename T, typename Acc, int VEC, int NCH, bool HAS_Y, bool FULL>
__global__ __launch_bounds__(kThreads) void resid_grad_kernel(
    int64_t n, int d, const T* __restrict__ X, int64_t ldx, const T* __restrict__ Y, int64_t incy,
    const double* __restrict__ beta, int lpr, double* __restrict__ partial, int ldp,
    const int* __restrict__ done) {
  if (done && *done) return;
  resid_grad<T, Acc, VEC, NCH, HAS_Y, FULL>(n, d, X, ldx, Y, incy, beta, lpr, partial, ldp);
}

// The pass of step t + 1 with the update of step t ahead of it: every block takes the
// update for itself (its partial rows, M and the iterates come from the caches), and
// block 0 writes it out, so the step is one launch.  Such a step is a chain of launches
// and cache latencies, not of bytes: whole float64 solves from their graphs, against a
// pass, an update and from 65 columns a sum of the rows as launches of their own:
// 16384 x 32 472 -> 338 us, 16384 x 64 578 -> 384, 16384 x 128 608 -> 573, 2^17 x 40
// 867 -> 716, 2^20 x 64 3800 -> 3655.
template <typename T, typename Acc, int VEC, int NCH, bool HAS_Y, bool FULL>
__global__ __launch_bounds__(kThreads) void step_grad_kernel(
    UpdateArgs u, int64_t n, int d, const T* __restrict__ X, int64_t ldx, const T* __restrict__ Y,
    int64_t incy, int lpr, double* __restrict__ partial, int ldp) {
  static_assert(kThreads == kStepThreads, "the update's split");
  __shared__ StepLds s_step;
  if (u.done && u.tol2 > 0.0) {
    // block 0 may raise it in this launch; a block that sees it has nothing left to do,
    // and all of it has to see the same
    __shared__ int s_done;
    if (threadIdx.x == 0) s_done = *u.done;
    __syncthreads();
    if (s_done) return;
  }
  if (step_in_block(u, blockIdx.x == 0, s_step)) return;
  resid_grad<T, Acc, VEC, NCH, HAS_Y, FULL>(n, d, X, ldx, Y, incy, s_step.beta, lpr,
                                             partial, ldp);
}

// g = scale * the sum of the partial rows (columns 0..d-1), rn = scale * the
// sum of their last column.  Sixteen columns per block: 64 row groups sum every
// 64th row, then each wave its four groups by lane exchange, then the waves
// in order.
constexpr int kSumThreads = 1024;
constexpr int kSumCols = 16;
__global__ __launch_bounds__(kSumThreads) void sum_rows_kernel(
    const double* __restrict__ part, int rows, int ldp, int d, double scale,
    double* __restrict__ g, double* __restrict__ rn) {
  __shared__ double s[kSumThreads / 64][kSumCols];
  const int c = threadIdx.x % kSumCols, rg = threadIdx.x / kSumCols;
  const int col = blockIdx.x * kSumCols + c;
  constexpr int kGroups = kSumThreads / kSumCols;
  double t = 0.0;
  if (col <= d) {
    int k = rg;
    for (; k + 3 * kGroups < rows; k += 4 * kGroups) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = part[(int64_t)(k + u * kGroups) * ldp + col];
#pragma unroll
      for (int u = 0; u < 4; ++u) t += v[u];
    }
    for (; k < rows; k += kGroups) t += part[(int64_t)k * ldp + col];
  }
  t += wave_xor(t, 16);
  t += wave_xor(t, 32);
  if ((threadIdx.x & 63) < kSumCols) s[threadIdx.x >> 6][c] = t;
  __syncthreads();
  if (threadIdx.x < kSumCols && col <= d) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kSumThreads / 64; ++w) v += s[w][c];
    if (col < d)
      g[col] = scale * v;
    else if (rn)
      rn[0] = scale * v;
  }
}

constexpr int kStepChunks = 4;  // chunks per lane that a pass of at most kStepD columns takes

template <typename T, typename Acc, int VEC, int NCH, bool FULL>
void launch_t(const ResidGradPlan& pl, const ResidGradArgs& a, hipStream_t s) {
  const T* X = static_cast<const T*>(a.X);
  const T* Y = static_cast<const T*>(a.Y);
  if constexpr (NCH <= kStepChunks) {
    if (a.step) {
      if (Y)
        step_grad_kernel<T, Acc, VEC, NCH, true, FULL><<<pl.blocks, kThreads, 0, s>>>(
            *a.step, a.n, a.d, X, a.ldx, Y, a.incy, pl.lpr, a.partial, pl.ldp);
      else
        step_grad_kernel<T, Acc, VEC, NCH, false, FULL><<<pl.blocks, kThreads, 0, s>>>(
            *a.step, a.n, a.d, X, a.ldx, Y, a.incy, pl.lpr, a.partial, pl.ldp);
      return;
    }
  }
  if (Y) {
    resid_grad_kernel<T, Acc, VEC, NCH, true, FULL><<<pl.blocks, kThreads, 0, s>>>(
        a.n, a.d, X, a.ldx, Y, a.incy, a.beta, pl.lpr, a.partial, pl.ldp, a.done);
  } else {
    resid_grad_kernel<T, Acc, VEC, NCH, false, FULL><<<pl.blocks, kThreads, 0, s>>>(
        a.n, a.d, X, a.ldx, Y, a.incy, a.beta, pl.lpr, a.partial, pl.ldp, a.done);
  }
}

template <typename T, typename Acc>
void launch_vec(const ResidGradPlan& pl, const ResidGradArgs& a, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  if (pl.vec == 1) {
    launch_t<T, Acc, 1, 1, false>(pl, a, s);
    return;
  }
  if (pl.full) {
    switch (pl.nch) {
      case 1: launch_t<T, Acc, V, 1, true>(pl, a, s); return;
      case 2: launch_t<T, Acc, V, 2, true>(pl, a, s); return;
      case 4: launch_t<T, Acc, V, 4, true>(pl, a, s); return;
      case 8: launch_t<T, Acc, V, 8, true>(pl, a, s); return;
      case 16: launch_t<T, Acc, V, 16, true>(pl, a, s); return;
    }
  } else {
    switch (pl.nch) {
      case 1: launch_t<T, Acc, V, 1, false>(pl, a, s); return;
      case 2: launch_t<T, Acc, V, 2, false>(pl, a, s); return;
      case 3: launch_t<T, Acc, V, 3, false>(pl, a, s); return;
      case 4: launch_t<T, Acc, V, 4, false>(pl, a, s); return;
      case 5: launch_t<T, Acc, V, 5, false>(pl, a, s); return;
      case 6: launch_t<T, Acc, V, 6, false>(pl, a, s); return;
      case 7: launch_t<T, Acc, V, 7, false>(pl, a, s); return;
      case 8: launch_t<T, Acc, V, 8, false>(pl, a, s); return;
    }
  }
  fail(SLSE_EUNSUPPORTED, "resid_grad: unsupported chunk count");
}

}  // namespace

ResidGradPlan plan_resid_grad(int64_t n, int d, slse_dtype storage, const void* X, int64_t ldx,
                              int grid_blocks, int capacity, int lpr_hint) {
  ResidGradPlan pl;
  const int es = (int)dtype_size(storage);
  const int vfull = 16 / es;
  // vectors at any element address; rows shorter than one take an element per lane
  pl.vec = d >= vfull ? vfull : 1;
  const int nvec = (int)ceil_div(d, pl.vec);
  // Four to eight elements per lane, lane groups a power of 2 up to a wave: a wave's
  // loads then cover whole rows side by side, and few rows still fill the chip.  Best or
  // within 3% of it from 4096 to 16 million rows of 16 to 512 columns in both types;
  // eight vectors per lane, in comparison: 16384 x 32 float64 11.6 -> 6.8 us (the
  // gradient with its sum), 2^21 x 32 float32 165 -> 49 us, 2^20 x 256 float32
  // 168 -> 162 us.
  int lpr = 1;
  while (lpr < 64 && lpr * 8 <= d) lpr *= 2;
  if (lpr_hint > 0) lpr = lpr_hint;
  if (const char* e = std::getenv("SLSE_RG_LPR")) lpr = std::atoi(e);
  lpr = std::max(1, std::min(64, lpr));
  while (lpr & (lpr - 1)) lpr &= lpr - 1;
  bool full_ok = pl.vec > 1 && is_pow2(nvec) && d % pl.vec == 0;
  if (const char* e = std::getenv("SLSE_RG_FULL")) full_ok = full_ok && std::atoi(e) != 0;
  // whole chunks: 1, 2, 4, 8 or 16 per lane; with a moved last chunk 1 to 8; one
  // element per lane below a vector
  const int most = pl.vec == 1 ? 1 : full_ok ? 16 : 8;
  while (lpr < 64 && ceil_div(nvec, lpr) > most) lpr *= 2;
  pl.nch = (int)ceil_div(nvec, lpr);
  if (pl.nch > most) fail(SLSE_EUNSUPPORTED, "resid_grad: d too large for this build");
  pl.lpr = lpr;
  pl.full = full_ok && (int64_t)pl.nch * lpr * pl.vec == d;
  pl.ldp = (int)round_up(d + 1, 8);
  const int rows_per_block_step = kWaves * (64 / lpr);
  const int bytes_per_vec = pl.vec * es;
  const int unroll = std::max(1, std::min(16, 256 / (pl.nch * bytes_per_vec)));
  // an override may choose another grid, never one above the capacity the
  // partial rows were allocated for
  int target = std::min(grid_blocks, capacity);
  if (const char* e = std::getenv("SLSE_RG_BLOCKS"))
    target = std::max(1, std::min(capacity, std::atoi(e)));
  int64_t want = ceil_div(std::max<int64_t>(n, 1), (int64_t)rows_per_block_step * unroll);
  pl.blocks = (int)std::max<int64_t>(1, std::min<int64_t>(want, target));
  return pl;
}

bool resid_grad_takes_step(const ResidGradPlan& pl, const UpdateArgs& u) {
  return step_fits(u.d, u.rows) && pl.blocks <= 512 && pl.nch <= kStepChunks;
}

void launch_resid_grad(const ResidGradPlan& pl, const ResidGradArgs& a, hipStream_t s) {
  if (pl.blocks > a.capacity_blocks)
    fail(SLSE_EINVAL, "resid_grad: plan exceeds the scratch capacity");
  if (a.step && (!resid_grad_takes_step(pl, *a.step) || a.step->d != a.d))
    fail(SLSE_EINVAL, "resid_grad: the update does not fit the pass");
  if (a.storage == SLSE_F64) {
    if (a.accum == SLSE_F64)
      launch_vec<double, double>(pl, a, s);
    else
      launch_vec<double, float>(pl, a, s);
  } else if (a.storage == SLSE_F32) {
    if (a.accum == SLSE_F64)
      launch_vec<float, double>(pl, a, s);
    else
      launch_vec<float, float>(pl, a, s);
  } else {
    fail(SLSE_EUNSUPPORTED, "resid_grad: storage must be F32 or F64");
  }
  SLSE_LAUNCH_CHECK();
}

void launch_sum_rows(const double* part, int rows, int ldp, int d, double scale, double* g,
                     double* rnorm2, hipStream_t s) {
  sum_rows_kernel<<<(int)ceil_div(d + 1, kSumCols), kSumThreads, 0, s>>>(part, rows, ldp, d, scale,
                                                                       g, rnorm2);
  SLSE_LAUNCH_CHECK();
}

}  // namespace slse
