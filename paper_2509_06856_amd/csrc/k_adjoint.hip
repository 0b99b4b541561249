// Fused rank-2 adjoint pass.  For L with dL/dbeta_hat = w and
// lambda = (X^T X)^{-1} w, differentiating the normal equations X^T X
// beta_hat = X^T Y (problem statement, Sec. 1) gives per row j
//     u_j = x_j . lambda,  r_j = y_j - x_j . beta_hat,
//     dY_j = u_j,          dX_j = r_j lambda^T - u_j beta_hat^T.
// One read of [x_j | y_j], one write of [dX_j | dY_j]; both dots accumulate in
// FP64.  Row split over lane groups as in the residual-gradient pass.
#include <algorithm>

#include "kernels.hpp"
#include "rng.hpp"

namespace slse {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// a vector of VEC elements whose address is a multiple of the element size
template <typename T, int VEC>
struct VecOf {
  typedef T type __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
};
template <typename T, int VEC>
using vec_of = typename VecOf<T, VEC>::type;

// VEC elements at p, any element address (16-byte vector loads/stores when VEC >
// 1), streamed past the caches
template <typename T, int VEC>
__device__ __forceinline__ void load_chunk(const T* __restrict__ p, T (&v)[VEC]) {
  if constexpr (VEC == 1) {
    v[0] = __builtin_nontemporal_load(p);
  } else {
    const vec_of<T, VEC> t = __builtin_nontemporal_load(reinterpret_cast<const vec_of<T, VEC>*>(p));
#pragma unroll
    for (int k = 0; k < VEC; ++k) v[k] = t[k];
  }
}
template <typename G, int VEC>
__device__ __forceinline__ void store_chunk(G* __restrict__ p, const G (&v)[VEC]) {
  if constexpr (VEC == 1) {
    __builtin_nontemporal_store(v[0], p);
  } else {
    vec_of<G, VEC> t;
#pragma unroll
    for (int k = 0; k < VEC; ++k) t[k] = v[k];
    __builtin_nontemporal_store(t, reinterpret_cast<vec_of<G, VEC>*>(p));
  }
}

// rows of [X|Y] a lane keeps in flight: about 128 bytes of X per lane
template <typename T, int VEC, int NCH>
constexpr int adjoint_unroll() {
  constexpr int u = 128 / (NCH * VEC * (int)sizeof(T));
  return u < 1 ? 1 : (u > 8 ? 8 : u);
}

// A row is split over `lpr` lanes, each holding NCH chunks of VEC columns
// (column (c lpr + l) VEC + k); a block handles tiles of UNROLL x (rows per
// block step) rows, every lane group keeping UNROLL rows in flight.  Rows of X and
// dX may start at any element.  Where d ends inside a chunk, the chunk is moved
// back to end with the row: its columns that another lane holds stay out of the
// dots and are written twice, with the same values.  Whole calls on float32 (lambda's
// first iterate and this pass): 2^20 x 101 628 -> 359 us, 2^20 x 256 with rows 259 apart
// 1214 -> 495 us (both took an element per lane), 2^20 x 256 535 -> 469 us (loads
// without a guard each).
template <typename T, typename G, int VEC, int NCH>
__global__ __launch_bounds__(kThreads) void adjoint_kernel(int64_t n, int d, const T* __restrict__ X,
                                                           int64_t ldx, const T* __restrict__ Y,
                                                           const double* __restrict__ beta,
                                                           const double* __restrict__ lambda,
                                                           int lpr, G* __restrict__ dX, int64_t lddx,
                                                           G* __restrict__ dY) {
  constexpr int UNROLL = adjoint_unroll<T, VEC, NCH>();
  // chunks that lie inside the row for every lane: all but the last where NCH is
  // the exact count, half of them where it is rounded up to a power of 2
  constexpr int kSure = NCH <= 4 ? NCH - 1 : NCH / 2;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int gpw = 64 / lpr;
  const int grp = lane / lpr;
  const int l = lane - grp * lpr;
  double b[NCH][VEC], lam[NCH][VEC];
  int col[NCH], at[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    col[c] = (c * lpr + l) * VEC;
    at[c] = min(col[c], d - VEC);
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      b[c][k] = beta[at[c] + k];
      lam[c][k] = lambda[at[c] + k];
    }
  }
  const int step = kWaves * gpw;  // rows per block step
  const int64_t tile = (int64_t)step * UNROLL;
  const int my = wave * gpw + grp;
  for (int64_t base = (int64_t)blockIdx.x * tile; base < n; base += (int64_t)gridDim.x * tile) {
    T x[UNROLL][NCH][VEC];
    double y[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      // past the end: the last row again, not stored
      const int64_t row = min(base + (int64_t)u * step + my, n - 1);
      const T* xr = X + row * ldx;
#pragma unroll
      for (int c = 0; c < kSure; ++c) load_chunk<T, VEC>(xr + at[c], x[u][c]);
      y[u] = Y ? (double)Y[row] : 0.0;
    }
    // the chunks that may lie past the row: lanes without columns stay idle
#pragma unroll
    for (int c = kSure; c < NCH; ++c) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
#pragma unroll
        for (int k = 0; k < VEC; ++k) x[u][c][k] = (T)0;
      if (col[c] < d) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
          const int64_t row = min(base + (int64_t)u * step + my, n - 1);
          load_chunk<T, VEC>(X + row * ldx + at[c], x[u][c]);
        }
      }
    }
    double d1[UNROLL], d2[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      double s1 = 0.0, s2 = 0.0;
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
          // (a sum kept, not a zero added: 0 times an infinite coefficient is NaN)
          const bool own = c < kSure || at[c] + k >= col[c];
          const double v = (double)x[u][c][k];
          s1 = own ? fma(v, b[c][k], s1) : s1;
          s2 = own ? fma(v, lam[c][k], s2) : s2;
        }
      d1[u] = s1;
      d2[u] = s2;
    }
    for (int m = lpr >> 1; m > 0; m >>= 1) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        d1[u] += wave_xor(d1[u], m);
        d2[u] += wave_xor(d2[u], m);
      }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t row = base + (int64_t)u * step + my;
      if (row >= n) continue;
      const double r = y[u] - d1[u];
      if (dX) {
        G* out = dX + row * lddx;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          if (c >= kSure && col[c] >= d) continue;
          G o[VEC];
#pragma unroll
          for (int k = 0; k < VEC; ++k) o[k] = (G)(r * lam[c][k] - d2[u] * b[c][k]);
          store_chunk<G, VEC>(out + at[c], o);
        }
      }
      if (dY && l == 0) dY[row] = (G)d2[u];
    }
  }
}

template <typename T, typename G, int VEC, int NCH>
void launch4(const AdjointArgs& a, int lpr, hipStream_t s) {
  const int64_t tile = (int64_t)kWaves * (64 / lpr) * adjoint_unroll<T, VEC, NCH>();
  const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(a.n, tile), 2048));
  adjoint_kernel<T, G, VEC, NCH><<<blocks, kThreads, 0, s>>>(
      a.n, a.d, static_cast<const T*>(a.X), a.ldx, static_cast<const T*>(a.Y), a.beta, a.lambda,
      lpr, static_cast<G*>(a.dX), a.lddx, static_cast<G*>(a.dY));
  SLSE_LAUNCH_CHECK();
}

template <typename T, typename G, int VEC>
void launch3(const AdjointArgs& a, hipStream_t s) {
  // lane groups of at most a wave, about four chunks per lane
  const int nvec = (int)ceil_div(a.d, VEC);
  int lpr = 1;
  while (lpr < 64 && lpr * 4 < nvec) lpr *= 2;
  const int nch = (int)ceil_div(nvec, lpr);
  if (nch <= 1)
    launch4<T, G, VEC, 1>(a, lpr, s);
  else if (nch <= 2)
    launch4<T, G, VEC, 2>(a, lpr, s);
  else if (nch <= 3)
    launch4<T, G, VEC, 3>(a, lpr, s);
  else if (nch <= 4)
    launch4<T, G, VEC, 4>(a, lpr, s);
  else if (nch <= 8)
    launch4<T, G, VEC, 8>(a, lpr, s);
  else if (nch <= 16)
    launch4<T, G, VEC, 16>(a, lpr, s);
  else
    fail(SLSE_EUNSUPPORTED, "adjoint: d too large for this library");
}

template <typename T, typename G>
void launch2(const AdjointArgs& a, hipStream_t s) {
  // 16-byte chunks, but for rows shorter than one, and for FP64 rows off the
  // 16-byte grid: two values a lane then gain nothing over one, whose lane groups fit
  // narrow rows better (whole calls on 2^20 x 33: 251 against 267 us, on 2^19 x 255
  // 550 against 552)
  constexpr int V = 16 / (int)sizeof(T);
  auto aligned = [](const void* p, int64_t ld, size_t es) {
    return p == nullptr || (reinterpret_cast<uintptr_t>(p) % 16 == 0 && (ld * (int64_t)es) % 16 == 0);
  };
  if (a.d < V || (sizeof(T) == 8 && !(a.d % V == 0 && aligned(a.X, a.ldx, sizeof(T)) &&
                                      aligned(a.dX, a.lddx, sizeof(G)))))
    launch3<T, G, 1>(a, s);
  else
    launch3<T, G, V>(a, s);
}

// ---------------------------------------------------------------------------
// Test hook: the counter streams as the device computes them.
// ---------------------------------------------------------------------------
__global__ void debug_stream_kernel(int what, uint64_t seed, int stream_id, int64_t aux,
                                    int64_t start, int64_t count, int64_t* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t x = (uint64_t)(start + i);
    switch (what) {
      case 0: {
        rng::Words w = rng::philox(x, (uint64_t)aux, 0, 0, seed, (uint64_t)stream_id);
        for (int k = 0; k < 4; ++k) out[4 * i + k] = (int64_t)w.w[k];
        break;
      }
      case 1: out[i] = (int64_t)rng::prp(x, seed, (uint64_t)stream_id, (int)aux); break;
      case 2: out[i] = (int64_t)rng::prp_inv(x, seed, (uint64_t)stream_id, (int)aux); break;
      case 3: out[i] = rng::rademacher(seed, x); break;
      case 4:
      case 5: {
        uint64_t bkt;
        int sg;
        rng::cs_hash(seed, x, (uint64_t)aux - 1, bkt, sg);
        out[i] = what == 4 ? (int64_t)bkt : sg;
        break;
      }
      default: {
        uint64_t bkt;
        int sg;
        rng::cs_hash_hat(seed, x, (uint64_t)aux, bkt, sg);
        out[i] = what == 6 ? (int64_t)bkt : sg;
        break;
      }
    }
  }
}

}  // namespace

void launch_adjoint(const AdjointArgs& a, hipStream_t s) {
  if (a.n <= 0) return;
  if (a.t == SLSE_F64 && a.gt == SLSE_F64)
    launch2<double, double>(a, s);
  else if (a.t == SLSE_F32 && a.gt == SLSE_F32)
    launch2<float, float>(a, s);
  else if (a.t == SLSE_F32 && a.gt == SLSE_F64)
    launch2<float, double>(a, s);
  else if (a.t == SLSE_F64 && a.gt == SLSE_F32)
    launch2<double, float>(a, s);
  else
    fail(SLSE_EUNSUPPORTED, "adjoint: dtype");
}

void launch_debug_stream(int what, uint64_t seed, int stream_id, int64_t aux, int64_t start,
                         int64_t count, int64_t* out, hipStream_t s) {
  if (count <= 0) return;
  const int blocks = (int)std::min<int64_t>(ceil_div(count, 256), 4096);
  debug_stream_kernel<<<blocks, 256, 0, s>>>(what, seed, stream_id, aux, start, count, out);
  SLSE_LAUNCH_CHECK();
}

}  // namespace slse
