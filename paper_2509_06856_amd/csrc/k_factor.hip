// Dense FP64 kernels behind slse_factor: the Hessian sketch
// H_hat = (S_hat X)^T S_hat X (Sec. 3) is applied through its triangular
// factor R (R^T R = H_hat; QR route of the implementation-details appendix).
//
//  gram        G = alpha A^T A, the upper tiles on the FP64 matrix cores
//  cholesky    R^T R = G together with Z = R^{-T}, one launch per 32 columns
//  gemm        Q = alpha A Z^T (a CholeskyQR pass) and small d x d products
// and M = (R^T R)^{-1} = Z^T Z, once more the Gram kernel.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kernels.hpp"

namespace slse {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// value of `v` held by lane `lane` (uniform), broadcast to the wave
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// ---------------------------------------------------------------------------
// FP64 products on the matrix cores (v_mfma_f64_16x16x4_f64: lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator r of lane l is
// C[4 r + l / 16][l % 16]).  A block of four waves computes an
// S x S tile (S = 32 MT), each wave MT x MT MFMA tiles, in steps of 32 k staged
// through LDS; the next step's loads are in flight during the products.
// Matrix products of the factor are small (d <= 1024), so what bounds them
// is latency: S = 32 where a product has few tiles, S = 64 where the tiles and
// the row splits fill the chip anyway (twice the products per LDS read).
// ---------------------------------------------------------------------------
constexpr int kKS = 32;  // k per step

template <int MT>
struct GemmLds {
  // row strides: 2 x stride = 8 and 32 banks mod 64, so that the 16 x 4 lanes
  // of an operand read fall into distinct banks
  double a[kKS][32 * MT + 16];
  double b[kKS][32 * MT + 16];
};

// acc += op(A)[i0 .., k] op(B)[k, j0 ..] over k in [kb0, kend), for PRE of pre A and pre B.
// TRA: A is stored k-major (A[k][i]), else i-major; TRB: B is stored j-major
// (B[j][k]), else k-major.  (PRE at compile time: behind a branch every thread waited for all
// its loads there, 300000 x 1 float32 306 -> 318 us; on the operands, among the products,
// 300000 x 200 float64 1030 -> 1165 us, on their way to LDS 1021.)
template <int MT, bool TRA, bool TRB, bool PRE, typename AP, typename BP>
__device__ __forceinline__ void mfma_tile(GemmLds<MT>& lds, AP __restrict__ A, int64_t lda,
                                          BP __restrict__ B, int64_t ldb, int64_t M, int64_t N,
                                          int64_t i0, int64_t j0, int64_t kb0, int64_t kend,
                                          double pre, f64x4 (&acc)[MT][MT]) {
  constexpr int S = 32 * MT;
  constexpr int kL = kKS * S / 256;  // entries of A and of B per thread per step
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int wr = (wave >> 1) * 16 * MT, wc = (wave & 1) * 16 * MT;
  double va[kL], vb[kL];
  unsigned oka = 0, okb = 0;
  // loads outside the matrices read a clamped, valid address and become zero
  // on their way to LDS, so none sits behind a branch
  auto fetch = [&](int64_t k0) {
    oka = okb = 0;
#pragma unroll
    for (int u = 0; u < kL; ++u) {
      const int e = t + 256 * u;
      const int ia = TRA ? e % S : e / kKS, ka = TRA ? e / S : e % kKS;
      const int64_t gi = i0 + ia, gk = k0 + ka;
      oka |= (unsigned)(gi < M && gk < kend) << u;
      const int64_t ci = min(gi, M - 1), ck = min(gk, kend - 1);
      va[u] = (double)(TRA ? A[ck * lda + ci] : A[ci * lda + ck]);
      const int jb = TRB ? e / kKS : e % S, kb = TRB ? e % kKS : e / S;
      const int64_t gj = j0 + jb, gq = k0 + kb;
      okb |= (unsigned)(gj < N && gq < kend) << u;
      const int64_t cj = min(gj, N - 1), cq = min(gq, kend - 1);
      vb[u] = (double)(TRB ? B[cj * ldb + cq] : B[cq * ldb + cj]);
    }
  };
  if (kb0 < kend) fetch(kb0);
  for (int64_t k0 = kb0; k0 < kend; k0 += kKS) {
#pragma unroll
    for (int u = 0; u < kL; ++u) {
      const int e = t + 256 * u;
      const int ia = TRA ? e % S : e / kKS, ka = TRA ? e / S : e % kKS;
      lds.a[ka][ia] = ((oka >> u) & 1) ? (PRE ? va[u] * pre : va[u]) : 0.0;
      const int jb = TRB ? e / kKS : e % S, kb = TRB ? e % kKS : e / S;
      lds.b[kb][jb] = ((okb >> u) & 1) ? (PRE ? vb[u] * pre : vb[u]) : 0.0;
    }
    __syncthreads();
    if (k0 + kKS < kend) fetch(k0 + kKS);
#pragma unroll
    for (int ks = 0; ks < kKS; ks += 4) {
      double a[MT], b[MT];
#pragma unroll
      for (int u = 0; u < MT; ++u) {
        a[u] = lds.a[ks + (lane >> 4)][wr + 16 * u + (lane & 15)];
        b[u] = lds.b[ks + (lane >> 4)][wc + 16 * u + (lane & 15)];
      }
#pragma unroll
      for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int v = 0; v < MT; ++v)
          acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
    }
    __syncthreads();
  }
}

// f(row, column, value) for every entry of this thread's accumulators
template <int MT, typename F>
__device__ __forceinline__ void for_acc(const f64x4 (&acc)[MT][MT], F&& f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = (wave >> 1) * 16 * MT, wc = (wave & 1) * 16 * MT;
#pragma unroll
  for (int u = 0; u < MT; ++u)
#pragma unroll
    for (int v = 0; v < MT; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        f(wr + 16 * u + 4 * r + (lane >> 4), wc + 16 * v + (lane & 15), acc[u][v][r]);
}

template <int MT>
__device__ __forceinline__ void clear_acc(f64x4 (&acc)[MT][MT]) {
#pragma unroll
  for (int u = 0; u < MT; ++u)
#pragma unroll
    for (int v = 0; v < MT; ++v) acc[u][v] = f64x4{0.0, 0.0, 0.0, 0.0};
}

// row and column tile of upper tile number `t` (column by column: (0,0),
// (0,1), (1,1), (0,2), ..)
__device__ __forceinline__ void upper_tile(int t, int& ti, int& tj) {
  tj = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while (tj * (tj + 1) / 2 > t) --tj;
  while ((tj + 1) * (tj + 2) / 2 <= t) ++tj;
  ti = t - tj * (tj + 1) / 2;
}

// One upper tile of G = alpha (pre A)^T (pre A) over the rows [kb0, kend) (pre = 1 unless
// PRE): written to both triangles of G, or without alpha to split slot `zpart` of `part`
// when there are several.
template <int MT, bool PRE, typename AP, typename GP, typename PP>
__device__ __forceinline__ void gram_tile(int d, double pre, double alpha, AP __restrict__ A, int64_t lda,
                                          GP __restrict__ G, int64_t ldg, PP __restrict__ part,
                                          int zpart, int tile, int64_t kb0, int64_t kend) {
  __shared__ GemmLds<MT> lds;
  int ti, tj;
  upper_tile(tile, ti, tj);
  const int i0 = ti * 32 * MT, j0 = tj * 32 * MT;
  f64x4 acc[MT][MT];
  clear_acc(acc);
  mfma_tile<MT, true, false, PRE>(lds, A, lda, A, lda, d, d, i0, j0, kb0, kend, pre, acc);
  for_acc(acc, [&](int r, int c, double v) {
    const int i = i0 + r, j = j0 + c;
    if (i >= d || j >= d) return;
    if (part) {
      part[((int64_t)zpart * d + i) * d + j] = v;
    } else {
      G[(int64_t)i * ldg + j] = alpha * v;
      if (ti != tj) G[(int64_t)j * ldg + i] = alpha * v;
    }
  });
}

template <int MT, bool PRE, typename T>
__global__ __launch_bounds__(256) void gram_kernel(int d, int64_t rows, double pre,
                                                   double alpha, const T* __restrict__ A,
                                                   int64_t lda, double* __restrict__ G, int64_t ldg,
                                                   double* __restrict__ part, int64_t kper) {
  const int64_t kb0 = (int64_t)blockIdx.y * kper;
  gram_tile<MT, PRE>(d, pre, alpha, A, lda, G, ldg, part, (int)blockIdx.y, (int)blockIdx.x, kb0,
                min(rows, kb0 + kper));
}

// G = alpha sum_s part[s] from the upper tiles of side S (splits summed in order)
template <typename GP, typename PP>
__device__ __forceinline__ void gram_reduce(int d, int S, int splits, double alpha,
                                            PP __restrict__ part, GP __restrict__ G, int64_t ldg) {
  const int64_t n = (int64_t)d * d;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / d), j = (int)(e % d);
    if (i / S > j / S) continue;  // below the upper tiles: written from its mirror
    double t = 0.0;
    for (int q = 0; q < splits; ++q) t += part[(int64_t)q * n + e];
    G[(int64_t)i * ldg + j] = alpha * t;
    if (i / S < j / S) G[(int64_t)j * ldg + i] = alpha * t;
  }
}

__global__ void gram_reduce_kernel(int d, int S, int splits, double alpha,
                                   const double* __restrict__ part, double* __restrict__ G,
                                   int64_t ldg) {
  gram_reduce(d, S, splits, alpha, part, G, ldg);
}

// C = alpha A op(B), one S x S tile per block, the column tiles of a row side by side on
// blockIdx.x (the other dimensions of a grid end at 65536 blocks: 2^21 rows of A);
// blockIdx.z picks one of two products of the same shape.
template <typename T>
struct GemmPair {
  const T* A[2];
  const double* B[2];
  double* C[2];
  int64_t ldc[2];
};

template <int MT, bool TRB, typename T>
__global__ __launch_bounds__(256) void gemm_kernel(int64_t M, int64_t N, int64_t K, double alpha,
                                                   GemmPair<T> p, int64_t lda, int64_t ldb) {
  __shared__ GemmLds<MT> lds;
  const int z = blockIdx.z;
  const unsigned nt = (unsigned)ceil_div(N, 32 * MT);
  const int64_t i0 = (int64_t)(blockIdx.x / nt) * 32 * MT, j0 = (int64_t)(blockIdx.x % nt) * 32 * MT;
  double* __restrict__ C = p.C[z];
  const int64_t ldc = p.ldc[z];
  f64x4 acc[MT][MT];
  clear_acc(acc);
  mfma_tile<MT, false, TRB, false>(lds, p.A[z], lda, p.B[z], ldb, M, N, i0, j0, 0, K, 1.0, acc);
  for_acc(acc, [&](int r, int c, double v) {
    if (i0 + r < M && j0 + c < N) C[(i0 + r) * ldc + j0 + c] = alpha * v;
  });
}

// ---------------------------------------------------------------------------
// Cholesky R^T R = G together with Z = R^{-T}, right-looking, 32 columns per
// launch.  Step k with pivot tile K: every block factors the 32 x 32 pivot tile
// itself (one wave, about 4 us: cheaper than another launch that hands the
// factor over), and one block per trailing tile (i, j), i > k, applies the
// step to it:
//   j >= i : G[i, j] -= P_i^T P_j,   P_c = R_KK^{-T} G[K, c] = R[K, c]
//   j <  k : W[i, j] -= P_i^T Z[K, j],   Z[K, j] = R_KK^{-T} W[K, j]
//   j == k : W[i, k]  = -P_i^T R_KK^{-T}
// W, the identity being eliminated along with G, lives in the tiles of G
// below the diagonal (each is first written, not read, at its column's step),
// so G is destroyed.  The blocks of the first trailing row (the last step: of
// a virtual one) write row K of R and of Z; nothing of row K of G is written
// during step k, and every trailing tile belongs to one block.
//
// A step is latency: 9.6 us at d = 512, of which (taken apart) 2.6 the launch and the loads,
// 4.3 the pivot tile and 2.9 the three products with their LDS round trips.  The
// 16 steps take 0.157 ms, against 2.37 + 0.69 ms of a one-block Cholesky and a
// row-wise inverse (slse_factor, 3072 x 512: 3.24 -> 0.24 ms; CholeskyQR3 of
// 1536 x 256: 3.08 -> 0.40 ms) and 0.37 ms of a blocked Gauss-Jordan inverse with
// two launches per 32 columns, which the solves took.
// ---------------------------------------------------------------------------
constexpr int kCB = 32;       // columns per step
constexpr int kCBs = kCB + 16;  // LDS row stride

// 1/sqrt(p) for p > 0: the hardware's estimate (24 bits) and one step of order
// three
__device__ __forceinline__ double rsqrt_f64(double p) {
  const double y = __builtin_amdgcn_rsq(p);
  const double e = fma(-(p * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// 32 x 32 product acc (one 16 x 16 tile per wave) += X Y with X[m][k] at
// X[m * sxm + k * sxk] and Y[k][n] at Y[k * kCBs + n]
__device__ __forceinline__ void tile_product(const double* X, int sxm, int sxk, const double* Y,
                                             double sign, f64x4& acc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = (wave >> 1) * 16, c0 = (wave & 1) * 16;
#pragma unroll
  for (int ks = 0; ks < kCB; ks += 4) {
    const int k = ks + (lane >> 4);
    const double a = sign * X[(r0 + (lane & 15)) * sxm + k * sxk];
    const double b = Y[k * kCBs + c0 + (lane & 15)];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
}

// Sixteen elimination steps on columns of 16 rows, one per lane (lanes 0..15:
// the pivot block A = U^T U); leaves U^{-T} times the columns.  What bounds it
// is the chain from one pivot to the next, so the steps eliminate without
// square roots (row b loses A[a][b] / p_a times row a: a broadcast, a reciprocal and
// two products per step) and the rows are scaled by p_a^{-1/2} afterwards.
// Takes pivots whose reciprocal and its products stay in the normal range and returns
// whether all were such: guarding every pivot would lengthen the chain, so where it
// returns false, the columns of no use, the caller runs eliminate16_any on them.
__device__ __forceinline__ bool eliminate16(double (&col)[16]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int a = 0; a < 16; ++a) {
    const double p = readlane_f64(col[a], a);
    double m[16];
#pragma unroll
    for (int b = a + 1; b < 16; ++b) m[b] = readlane_f64(col[a], b);
    double inv = __builtin_amdgcn_rcp(p);  // 24 bits; one step of order three
    const double e = fma(-p, inv, 1.0);
    inv = fma(inv, fma(e, e, e), inv);
    const double w = col[a] * inv;
#pragma unroll
    for (int b = a + 1; b < 16; ++b) col[b] = fma(-m[b], w, col[b]);
  }
  // lane a < 16 holds p_a
  double p = 1.0;
#pragma unroll
  for (int a = 0; a < 16; ++a) p = lane == a ? col[a] : p;
  if (__ballot(!(p >= 0x1p-1000 && p <= 0x1p1000))) return false;
  const double y = rsqrt_f64(p);
  const double h = p * y;
  const double root = fma(0.5 * y, fma(-h, h, p), h);
#pragma unroll
  for (int a = 0; a < 16; ++a) col[a] = lane == a ? root : col[a] * readlane_f64(y, a);
  return true;
}

// The same for any pivots, on columns in LDS (column l at C[a * kCBs + l], l < 48; one
// wave): a pivot's reciprocal is its mantissa's and two powers of 2, so that each operand
// of a product stays near the square root of its own diagonal entry, and a bad pivot (not
// positive and finite) counts as 1, so that what it does not touch is factored as without
// it.  Returns c0 + a + 1 of the first bad pivot a, else 0.  Rare, so short code (a second
// unrolled form in registers cost every step 0.3 us: 132 VGPRs, twice the code).
__device__ __forceinline__ int eliminate16_any(double* C, int c0) {
  const int lane = threadIdx.x & 63;
  double* mine = C + min(lane, 47);  // the lanes past 48 repeat column 47
  int bad = 0;
#pragma unroll 1
  for (int a = 0; a < 16; ++a) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double p = C[a * kCBs + a];
    if (!(p > 0.0 && p <= 1.7976931348623157e308)) {
      if (!bad) bad = c0 + a + 1;
      p = 1.0;
    }
    int x;
    const double mant = frexp(p, &x);
    const double w = ldexp(mine[a * kCBs], -(x >> 1)) / mant;
#pragma unroll 1
    for (int b = a + 1; b < 16; ++b)
      mine[b * kCBs] = fma(-ldexp(C[a * kCBs + b], (x >> 1) - x), w, mine[b * kCBs]);
    // row a is not read by the others any more
    const double root = sqrt(p);
    const double r = mine[a * kCBs] * (1.0 / root);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    mine[a * kCBs] = lane == a ? root : r;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return bad;
}

// One wave factors the 32 x 32 pivot tile D (rows of kCBs doubles in LDS): R_KK
// to Rs and R_KK^{-T} over D.  Two halves of 16 columns, so that the cross
// term is eight matrix-core products instead of 256 broadcast multipliers:
//   [A11 A12 | I]  ->  R11, R12, Z11             (lanes 0..15, 16..31, 32..47)
//   T = A22 - R12^T R12,   W = -R12^T Z11
//   [T | W | I]    ->  R22, Z21, Z22
// Returns k0 + a + 1 of the first bad pivot a, or 0.
__device__ __forceinline__ int pivot_tile(double* D, double* Rs, int k0) {
  const int lane = threadIdx.x & 63;
  const int c = lane & 15, q = lane >> 4;
  // selections by per-lane integers, so that they stay selections (a
  // condition of several parts becomes branches around every register: 14 us a
  // step instead of 9.8)
  const bool data = q < 2;
  const int one = q == 2 ? c : -1;  // the row of the identity column's 1
  const unsigned keep = q == 0   ? (2u << c) - 1  // rows kept of this lane's column
                        : q == 1 ? 0xffffu
                        : q == 2 ? 0x10000u - (1u << c)
                                 : 0u;
  double col[16];
  // the columns from `from`, eliminated; the lanes past 32 read a valid column and
  // replace it.  `work`: 16 rows of LDS that hold nothing yet
  auto eliminate = [&](const double* from, double* work, int c0) {
#pragma unroll
    for (int a = 0; a < 16; ++a) {
      const double v = from[a * kCBs];
      const double id = a == one ? 1.0 : 0.0;
      col[a] = data ? v : id;
    }
    if (eliminate16(col)) return 0;
    if (q < 3)
#pragma unroll 1
      for (int a = 0; a < 16; ++a)
        work[a * kCBs + lane] = data ? from[a * kCBs] : a == one ? 1.0 : 0.0;
    const int bad = eliminate16_any(work, c0);
#pragma unroll
    for (int a = 0; a < 16; ++a) col[a] = work[a * kCBs + min(lane, 47)];
    return bad;
  };
  f64x4 T;  // A22 in the accumulator layout
#pragma unroll
  for (int r = 0; r < 4; ++r) T[r] = D[(16 + 4 * r + q) * kCBs + 16 + c];
  const int bad0 = eliminate(D + (lane & 31), Rs, k0);
  // R11 | R12 to Rs, Z11 to the upper left of D, zeros to its upper right
  {
    double* out = data ? Rs + lane : D + (lane - 32);
#pragma unroll
    for (int a = 0; a < 16; ++a) out[a * kCBs] = (keep >> a) & 1 ? col[a] : 0.0;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  f64x4 W{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < 16; ks += 4) {
    const double r12 = Rs[(ks + q) * kCBs + 16 + c];  // (R12^T)[m][k] and R12[k][n] alike
    const double z11 = D[(ks + q) * kCBs + c];
    T = __builtin_amdgcn_mfma_f64_16x16x4f64(-r12, r12, T, 0, 0, 0);
    W = __builtin_amdgcn_mfma_f64_16x16x4f64(-r12, z11, W, 0, 0, 0);
  }
  // [W | T] through the lower half of D, back as columns
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    D[(16 + 4 * r + q) * kCBs + c] = W[r];
    D[(16 + 4 * r + q) * kCBs + 16 + c] = T[r];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int bad1 = eliminate(D + 16 * kCBs + (q == 0 ? 16 + c : c), Rs + 16 * kCBs, k0 + 16);
  // R22 to Rs (zeros left of it), Z21 | Z22 to the lower half of D
  {
    double* out = q == 0 ? Rs + 16 + c : q == 1 ? D + c : q == 2 ? D + 16 + c : Rs + c;
#pragma unroll
    for (int a = 0; a < 16; ++a) out[(16 + a) * kCBs] = (keep >> a) & 1 ? col[a] : 0.0;
  }
  return bad0 ? bad0 : bad1;
}

template <typename DP, typename RP, typename IP>
__device__ __forceinline__ void chol_step(int d, int k, DP __restrict__ G, RP __restrict__ R,
                                          int64_t ldr, DP __restrict__ Z, IP __restrict__ info,
                                          int j, int row) {
  __shared__ double Ds[kCB * kCBs];  // pivot tile, then R_KK^{-T}
  __shared__ double Rs[kCB * kCBs];  // R_KK (head blocks of column k)
  __shared__ double Gi[kCB * kCBs];  // G[K, i], then P_i
  __shared__ double Gj[kCB * kCBs];  // G[K, j] or W[K, j], then P_j or Z[K, j]
  const int nb = (int)ceil_div(d, kCB);
  const int i = k + 1 + row;
  const bool head = row == 0;
  const bool trail = i < nb;
  if (j > k && j < i) return;  // below the diagonal of the trailing part (uniform)
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int k0 = k * kCB, i0 = i * kCB, j0 = j * kCB;
  constexpr int kL = kCB * kCB / 256;
  // all of the block's loads at once, from clamped addresses
  double vd[kL], vi[kL], vj[kL];
#pragma unroll
  for (int u = 0; u < kL; ++u) {
    const int e = t + 256 * u;
    const int a = e / kCB, c = e % kCB;
    const int64_t rk = (int64_t)min(k0 + a, d - 1) * d;
    vd[u] = G[rk + min(k0 + c, d - 1)];
    vi[u] = G[rk + min(i0 + c, d - 1)];
    vj[u] = G[rk + min(j0 + c, d - 1)];
  }
  const int r0 = (wave >> 1) * 16, c0 = (wave & 1) * 16;
  f64x4 acc;  // this wave's 16 x 16 tile of (i, j)
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int gi = i0 + r0 + 4 * r + (lane >> 4), gj = j0 + c0 + (lane & 15);
    const double v = G[(int64_t)min(gi, d - 1) * d + min(gj, d - 1)];
    acc[r] = (j != k && trail && gi < d && gj < d) ? v : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kL; ++u) {
    const int e = t + 256 * u;
    const int a = e / kCB, c = e % kCB;
    const bool rowok = k0 + a < d;
    // the pivot tile is padded with the identity past d
    Ds[a * kCBs + c] = rowok && k0 + c < d ? vd[u] : (a == c ? 1.0 : 0.0);
    Gi[a * kCBs + c] = rowok && i0 + c < d ? vi[u] : 0.0;
    Gj[a * kCBs + c] = rowok && j0 + c < d ? vj[u] : 0.0;
  }
  __syncthreads();
  if (wave == 0) {
    const int bad = pivot_tile(Ds, Rs, k0);
    if (lane == 0 && head && j == k && bad) {
      if (*info == 0) *info = bad;
    }
  }
  __syncthreads();
  // P_i, and P_j or Z[K, j] (for j == k it is R_KK^{-T} itself)
  f64x4 pi{0.0, 0.0, 0.0, 0.0}, pj{0.0, 0.0, 0.0, 0.0};
  if (trail) tile_product(Ds, kCBs, 1, Gi, 1.0, pi);
  if (j != k) tile_product(Ds, kCBs, 1, Gj, 1.0, pj);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int o = (r0 + 4 * r + (lane >> 4)) * kCBs + c0 + (lane & 15);
    Gi[o] = pi[r];
    Gj[o] = j == k ? Ds[o] : pj[r];
  }
  __syncthreads();
  if (head) {
#pragma unroll
    for (int u = 0; u < kL; ++u) {
      const int e = t + 256 * u;
      const int a = e / kCB, c = e % kCB;
      if (k0 + a >= d || j0 + c >= d) continue;
      const int64_t gr = k0 + a, gc = j0 + c;
      const double p = Gj[a * kCBs + c];
      if (R) R[gr * ldr + gc] = j > k ? p : j == k ? Rs[a * kCBs + c] : 0.0;
      Z[gr * d + gc] = j > k ? 0.0 : p;
    }
  }
  if (!trail) return;
  tile_product(Gi, 1, kCBs, Gj, -1.0, acc);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int gi = i0 + r0 + 4 * r + (lane >> 4), gj = j0 + c0 + (lane & 15);
    if (gi < d && gj < d) G[(int64_t)gi * d + gj] = acc[r];
  }
}

__global__ __launch_bounds__(256) void chol_step_kernel(int d, int k, double* __restrict__ G,
                                                        double* __restrict__ R, int64_t ldr,
                                                        double* __restrict__ Z,
                                                        int* __restrict__ info) {
  chol_step(d, k, G, R, ldr, Z, info, (int)blockIdx.x, (int)blockIdx.y);
}

// ---------------------------------------------------------------------------
// The same for the jobs of a batch.
// ---------------------------------------------------------------------------
// G = scale (pre A)^T (pre A) of every job (blockIdx.z = job x splits + split): with splits > 1
// each split sums its share of the rows into the job's partial slot
template <typename T>
__global__ __launch_bounds__(256) void gram_batched_kernel(const FactorJob* __restrict__ jobs,
                                                           int splits) {
  const FactorJob jb = jobs[blockIdx.z / splits];
  const int sp = blockIdx.z % splits;
  const int nt = (int)ceil_div(jb.d, 32);
  if ((int)blockIdx.x >= nt * (nt + 1) / 2) return;
  const int64_t kper = round_up(ceil_div(jb.rows, (int64_t)splits), kKS);
  const int64_t kb0 = sp * kper;
  gram_tile<1, sizeof(T) == 8>(jb.d, jb.pre, jb.scale, gptr(static_cast<const T*>(jb.A)), jb.lda, gptr(jb.G), jb.d,
               splits > 1 ? gptr(jb.part) : nullptr, sp, (int)blockIdx.x, kb0,
               min(jb.rows, kb0 + kper));
}

__global__ void gram_reduce_batched_kernel(const FactorJob* __restrict__ jobs, int splits) {
  const FactorJob jb = jobs[blockIdx.y];
  gram_reduce(jb.d, 32, splits, jb.scale, gptr((const double*)jb.part), gptr(jb.G), jb.d);
}

__global__ __launch_bounds__(256) void chol_step_batched_kernel(const FactorJob* __restrict__ jobs,
                                                                int k) {
  const FactorJob jb = jobs[blockIdx.z];
  const int nb = (int)ceil_div(jb.d, kCB);
  if (k >= nb || (int)blockIdx.x >= nb || (int)blockIdx.y >= max(1, nb - k - 1)) return;
  chol_step(jb.d, k, gptr(jb.G), gptr((double*)nullptr), 0, gptr(jb.Z), jb.info, (int)blockIdx.x,
            (int)blockIdx.y);
}

// M = Z^T Z of every job
__global__ __launch_bounds__(256) void inverse_batched_kernel(const FactorJob* __restrict__ jobs) {
  const FactorJob jb = jobs[blockIdx.z];
  const int nt = (int)ceil_div(jb.d, 32);
  if ((int)blockIdx.x >= nt * (nt + 1) / 2) return;
  gram_tile<1, false>(jb.d, 1.0, 1.0, gptr((const double*)jb.Z), jb.d, gptr(jb.M), jb.d,
               (SLSE_GLOBAL double*)nullptr, 0, (int)blockIdx.x, 0, jb.d);
}

// G += coef trace(G) I (one block): the diagonal shift of shifted CholeskyQR
__global__ __launch_bounds__(256) void shift_diag_kernel(int d, double* __restrict__ G, double coef) {
  __shared__ double red[256];
  double t = 0.0;
  for (int i = threadIdx.x; i < d; i += 256) t += G[(int64_t)i * d + i];
  red[threadIdx.x] = t;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double shift = coef * red[0];
  for (int i = threadIdx.x; i < d; i += 256) G[(int64_t)i * d + i] += shift;
}

}  // namespace

void launch_shift_diag(int d, double* G, double coef, hipStream_t s) {
  shift_diag_kernel<<<1, 256, 0, s>>>(d, G, coef);
  SLSE_LAUNCH_CHECK();
}

// Row splits and tile of the Gram kernel: about 512 blocks of at least 128 rows.
struct GramShape {
  bool wide;  // 64 x 64 tiles
  int tiles, splits;
  int64_t kper;
};
GramShape gram_shape(int64_t rows, int64_t d) {
  GramShape g;
  g.wide = d > 192;  // 64-wide tiles leave too few blocks below (10 upper tiles at d = 256)
  const int64_t nt = ceil_div(d, g.wide ? 64 : 32);
  g.tiles = (int)(nt * (nt + 1) / 2);
  int64_t sp = std::max<int64_t>(1, 512 / g.tiles);
  sp = std::min<int64_t>({sp, std::max<int64_t>(1, rows / 128), 32});
  g.kper = sp > 1 ? round_up(ceil_div(rows, sp), kKS) : std::max<int64_t>(rows, 1);
  g.splits = (int)std::max<int64_t>(1, ceil_div(rows, g.kper));
  return g;
}

void gram_scale(double scale, slse_dtype at, double* pre, double* rest) {
  *pre = 1.0;
  *rest = scale;
  if (at == SLSE_F32 || !(scale > 0.0) || !std::isfinite(scale)) return;
  int e;
  const double f = std::frexp(scale, &e);  // scale = f 2^e, f in [1/2, 1)
  const int k = (e - 1) >> 1;              // scale / 4^k in [1, 4)
  *pre = std::ldexp(1.0, k);
  *rest = std::ldexp(f, e - 2 * k);
}

size_t gram_scratch_doubles(int64_t rows, int64_t d) {
  const GramShape g = gram_shape(rows, d);
  return g.splits > 1 ? (size_t)g.splits * d * d : 0;
}

void launch_gram(int64_t rows, int d, double alpha, const void* A, int64_t lda, slse_dtype at,
                 double* G, int64_t ldg, double* scratch, size_t scratch_doubles, hipStream_t s) {
  if (rows <= 0 || d <= 0) return;
  GramShape g = gram_shape(rows, d);
  if (g.splits > 1 && (!scratch || scratch_doubles < (size_t)g.splits * d * d)) {
    g.splits = 1;
    g.kper = rows;
  }
  double* part = g.splits > 1 ? scratch : nullptr;
  double pre;
  gram_scale(alpha, at, &pre, &alpha);
  const dim3 grid((unsigned)g.tiles, (unsigned)g.splits);
  auto go = [&](auto* a, auto scaled) {
    constexpr bool PRE = decltype(scaled)::value;
    if (g.wide)
      gram_kernel<2, PRE><<<grid, 256, 0, s>>>(d, rows, pre, alpha, a, lda, G, ldg, part, g.kper);
    else
      gram_kernel<1, PRE><<<grid, 256, 0, s>>>(d, rows, pre, alpha, a, lda, G, ldg, part, g.kper);
  };
  if (at == SLSE_F32)
    go(static_cast<const float*>(A), std::false_type{});
  else if (pre == 1.0)
    go(static_cast<const double*>(A), std::false_type{});
  else
    go(static_cast<const double*>(A), std::true_type{});
  SLSE_LAUNCH_CHECK();
  if (g.splits > 1) {
    const int blocks = (int)std::min<int64_t>(ceil_div((int64_t)d * d, 256), 4096);
    gram_reduce_kernel<<<blocks, 256, 0, s>>>(d, g.wide ? 64 : 32, g.splits, alpha, part, G, ldg);
    SLSE_LAUNCH_CHECK();
  }
}

void launch_times_inverse(int64_t rows, int d, double alpha, const void* A, int64_t lda,
                          slse_dtype at, const double* Z, double* Q, hipStream_t s) {
  if (rows <= 0 || d <= 0) return;
  const dim3 grid((unsigned)(ceil_div(d, 32) * ceil_div(rows, 32)));
  if (at == SLSE_F32) {
    const GemmPair<float> p{{static_cast<const float*>(A), nullptr}, {Z, nullptr}, {Q, nullptr},
                              {d, d}};
    gemm_kernel<1, true><<<grid, 256, 0, s>>>(rows, d, d, alpha, p, lda, d);
  } else {
    const GemmPair<double> p{{static_cast<const double*>(A), nullptr}, {Z, nullptr}, {Q, nullptr},
                              {d, d}};
    gemm_kernel<1, true><<<grid, 256, 0, s>>>(rows, d, d, alpha, p, lda, d);
  }
  SLSE_LAUNCH_CHECK();
}

void launch_two_products(int d, const double* A0, const double* B0, double* C0, int64_t ldc0,
                         const double* A1, const double* B1, double* C1, int64_t ldc1,
                         hipStream_t s) {
  if (d <= 0) return;
  const GemmPair<double> p{{A0, A1}, {B0, B1}, {C0, C1}, {ldc0, ldc1}};
  const unsigned nt = (unsigned)ceil_div(d, 32);
  gemm_kernel<1, false><<<dim3(nt * nt, 1, 2), 256, 0, s>>>(d, d, d, 1.0, p, d, d);
  SLSE_LAUNCH_CHECK();
}

void launch_cholesky(int d, double* G, double* R, int64_t ldr, double* Z, int* info,
                     hipStream_t s) {
  const int nb = (int)ceil_div(d, kCB);
  for (int k = 0; k < nb; ++k) {
    chol_step_kernel<<<dim3((unsigned)nb, (unsigned)std::max(1, nb - k - 1)), 256, 0, s>>>(
        d, k, G, R, ldr, Z, info);
    SLSE_LAUNCH_CHECK();
  }
}

int factor_batched_splits(int64_t rows_max) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(8, rows_max / 256));
}

void launch_factor_batched(const FactorJob* jobs, int B, int dmax, int64_t rows_max,
                           slse_dtype at, hipStream_t s) {
  if (B <= 0) return;
  if (dmax > 512) fail(SLSE_EUNSUPPORTED, "cholesky: d > 512 not supported by this library");
  if (B > 65535) fail(SLSE_EUNSUPPORTED, "factor: too many batched jobs");
  const int splits = factor_batched_splits(rows_max);
  if ((int64_t)B * splits > 65535) fail(SLSE_EUNSUPPORTED, "factor: too many batched jobs");
  const unsigned nb = (unsigned)ceil_div(dmax, kCB);
  const unsigned upper = nb * (nb + 1) / 2;
  const dim3 gg(upper, 1, (unsigned)(B * splits));
  if (at == SLSE_F32)
    gram_batched_kernel<float><<<gg, 256, 0, s>>>(jobs, splits);
  else
    gram_batched_kernel<double><<<gg, 256, 0, s>>>(jobs, splits);
  SLSE_LAUNCH_CHECK();
  if (splits > 1) {
    const unsigned rb = (unsigned)std::min<int64_t>(ceil_div((int64_t)dmax * dmax, 256), 256);
    gram_reduce_batched_kernel<<<dim3(rb, (unsigned)B), 256, 0, s>>>(jobs, splits);
    SLSE_LAUNCH_CHECK();
  }
  for (unsigned k = 0; k < nb; ++k) {
    chol_step_batched_kernel<<<dim3(nb, std::max(1u, nb - k - 1), (unsigned)B), 256, 0, s>>>(jobs,
                                                                                            (int)k);
    SLSE_LAUNCH_CHECK();
  }
  inverse_batched_kernel<<<dim3(upper, 1, (unsigned)B), 256, 0, s>>>(jobs);
  SLSE_LAUNCH_CHECK();
}

}  // namespace slse
