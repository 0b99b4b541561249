// Device parts of the M-IHS update that its own kernels and the residual-gradient
// kernel that starts with an update share.
#pragma once

#include "kernels.hpp"

namespace slse {

// the estimate of a step from its last sums: gp = g . Mg, pp = ||Mg||^2,
// bb = ||beta_{t+1}||^2; whether it ends the iteration
__device__ __forceinline__ bool step_ends(const UpdateArgs& a, double gp, double pp, double bb,
                                          double& est, bool& finite) {
  est = bb > 0.0 ? sqrt(pp / bb) : sqrt(pp);
  finite = isfinite(gp) && isfinite(pp) && isfinite(bb);
  return a.done && a.tol2 > 0.0 && (!finite || est * est <= a.tol2);
}
__device__ __forceinline__ void finish_step(const UpdateArgs& a, double gp, double pp, double bb) {
  double est;
  bool finite;
  const bool ends = step_ends(a, gp, pp, bb, est, finite);
  if (a.sur_out) a.sur_out[0] = est;
  if (!finite && a.status) atomicExch(a.status, 1);
  if (ends) atomicExch(a.done, 1);
}

// The updates that every block of a pass takes for itself: d columns and a sum of `rows`
// partial rows.  Each block reads M and the rows, up to 384 KB here (128 columns; 288 KB
// at 64); twice the width would be 1 MB, more than the launches that it saves.  Of 48 columns and 512 rows, 256
// rows as the limit was slower (2^18 x 48 float64 solve 1191 and 1227 us); wider problems
// have their rows summed first from 257 on.
constexpr int kStepD = 128;
constexpr int kStepThreads = 256;
__host__ __device__ inline bool step_fits(int d, int rows) {
  return d <= 64 ? rows <= 512 : d <= kStepD && rows <= 256;
}

struct StepLds {
  double p[kStepThreads][2];
  double g[kStepD];
  double sum[3][kStepD];
  double beta[kStepD];
  int end;
};

// The update of one step of at most D columns by a block of 256 threads, beta_{t+1} left
// in s.beta; block 0 alone (`lead`) writes it and the estimate out.  Returns whether the
// iteration ends here, the same in every block.  Sums run in a fixed order.
template <int D>
__device__ __forceinline__ bool step_of(const UpdateArgs& a, bool lead, StepLds& s) {
  constexpr int KQ = D / 8, RQ = D / 32;
  const int d = a.d;
  // eight lanes per row of M; its rows and the iterates are on their way meanwhile
  const int r0 = threadIdx.x >> 3, q = threadIdx.x & 7;
  double m[RQ][KQ], bi[RQ], bp[RQ];
#pragma unroll
  for (int j = 0; j < RQ; ++j) {
    const int i = r0 + 32 * j;
    const bool in = i < d;
    bi[j] = in ? a.beta[i] : 0.0;
    bp[j] = in ? a.beta_prev[i] : 0.0;
#pragma unroll
    for (int k = 0; k < KQ; ++k)
      m[j][k] = in && q + 8 * k < d ? a.M[(int64_t)i * a.ldm + q + 8 * k] : 0.0;
  }
  // 2^lc pairs of columns x 256 / 2^lc row groups, each summing every such row (the
  // rows are padded to whole pairs)
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  int lc = 0;
  while ((2 << lc) < d) ++lc;
  const int groups = kStepThreads >> lc;
  const int c = 2 * (threadIdx.x & ((1 << lc) - 1)), rg = threadIdx.x >> lc;
  f64x2 t = {0.0, 0.0};
  if (c < d) {
    const double* part = a.part + c;
    auto row = [&](int k) { return *reinterpret_cast<const f64x2*>(part + (int64_t)k * a.ldp); };
    constexpr int U = 16;
    int k = rg;
    for (; k + (U - 1) * groups < a.rows; k += U * groups) {
      f64x2 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = row(k + u * groups);
#pragma unroll
      for (int u = 0; u < U; ++u) t += v[u];
    }
    for (; k + 3 * groups < a.rows; k += 4 * groups) {
      f64x2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = row(k + u * groups);
#pragma unroll
      for (int u = 0; u < 4; ++u) t += v[u];
    }
    for (; k < a.rows; k += groups) t += row(k);
  }
  s.p[threadIdx.x][0] = t[0];
  s.p[threadIdx.x][1] = t[1];
  for (int k = threadIdx.x; k < kStepD; k += kStepThreads)
    for (int e = 0; e < 3; ++e) s.sum[e][k] = 0.0;
  __syncthreads();
  if ((int)threadIdx.x < d) {
    double v = 0.0;
    for (int k = 0; k < groups; ++k) v += s.p[(k << lc) + (threadIdx.x >> 1)][threadIdx.x & 1];
    double g = a.scale * v;
    if (a.w) g += a.w[threadIdx.x * a.incw];
    s.g[threadIdx.x] = g;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < RQ; ++j) {
    const int i = r0 + 32 * j;
    double p = 0.0;
#pragma unroll
    for (int k = 0; k < KQ; ++k) p = fma(m[j][k], q + 8 * k < d ? s.g[q + 8 * k] : 0.0, p);
    for (int x = 1; x < 8; x <<= 1) p += wave_xor(p, x);
    if (q == 0 && i < d) {
      const double bn = bi[j] + a.mu * p + a.eta * (bi[j] - bp[j]);
      s.beta[i] = bn;
      s.sum[0][i] = s.g[i] * p;
      s.sum[1][i] = p * p;
      s.sum[2][i] = bn * bn;
      if (lead) {
        a.beta_next[i] = bn;
        if (a.beta_out) a.beta_out[i] = bn;
        if (a.traj_row) a.traj_row[i] = bn;
      }
    }
  }
  __syncthreads();
  const bool tested = a.done && a.tol2 > 0.0;
  if (!lead && !tested) return false;
  if (threadIdx.x < 64) {
    double e[3];
    for (int k = 0; k < 3; ++k) {
      e[k] = s.sum[k][threadIdx.x] + s.sum[k][threadIdx.x + 64];
      for (int x = 32; x > 0; x >>= 1) e[k] += wave_xor(e[k], x);
    }
    if (threadIdx.x == 0) {
      double est;
      bool finite;
      s.end = step_ends(a, e[0], e[1], e[2], est, finite);
      if (lead) finish_step(a, e[0], e[1], e[2]);
    }
  }
  if (!tested) return false;
  __syncthreads();
  return s.end != 0;
}

__device__ __forceinline__ bool step_in_block(const UpdateArgs& a, bool lead, StepLds& s) {
  if (a.d <= 32) return step_of<32>(a, lead, s);
  if (a.d <= 64) return step_of<64>(a, lead, s);
  return step_of<128>(a, lead, s);
}

}  // namespace slse
