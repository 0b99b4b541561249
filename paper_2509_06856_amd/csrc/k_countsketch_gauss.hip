// CountSketch and Gaussian sketches of [X|Y] (Sec. 1.2; CountSketch as the
// alternative sketching matrix of Sec. 5.4).
//
// CountSketch: column j of S_K has the single entry s(j) in row h(j), so
// S_K [X|Y] adds s(j) [x_j | y_j] into bucket h(j).  Instead of scattering
// rows with float atomics, the rows are first listed per bucket (integer
// counts that give each row its rank, an exclusive scan, each row's index with
// its sign folded in placed by rank), and each output row is then gathered: a
// lane group per bucket of the largest level (m_K buckets, a few rows each) and
// several waves per bucket of the Hessian sketch (r buckets, about N/r rows
// each; their partial rows are added in a fixed order).  Smaller levels use the
// bucket h(j) mod m_i, so level i is level i+1 folded in halves: A_i[k] =
// sum_{t = k mod m_i} A_{i+1}[t].  Lists are put in increasing row order, so a
// sketch has the same bits on every run.
//
// Gaussian: A = G [X|Y] with G_kj iid N(0, 1) drawn on the fly (Philox block
// (j, k >> 3) -> four Box-Muller pairs), multiplied on the matrix cores with
// the N rows split over blocks; partial tiles are summed in split order by a
// second kernel.  FP64 data is multiplied and accumulated in FP64, FP32 data in
// FP32, or, on request, rounded to BF16 and accumulated in FP32.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "rng.hpp"

namespace slse {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

template <typename T>
__global__ void fill_kernel(T* __restrict__ p, int64_t rows, int64_t cols, int64_t ld) {
  const int64_t n = rows * cols;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / cols, c = e % cols;
    p[i * ld + c] = (T)0;
  }
}

constexpr int kHistLds = 8192;  // Hessian buckets counted in a wave's LDS up to this many

// The largest level's rows in their buckets: every row's bucket (complemented
// for a negative sign) and its arrival number there, which the count's atomic
// returns anyway; the list is then placed without drawing the hash or an
// atomic again (2^20 rows: count and fill 122 -> 62 us).
__global__ __launch_bounds__(kThreads) void cs_count_rank_kernel(int64_t n, uint64_t seed,
                                                                 uint64_t mK_mask,
                                                                 int* __restrict__ cntK,
                                                                 int* __restrict__ keys,
                                                                 int* __restrict__ rank) {
  for (int64_t j = blockIdx.x * (int64_t)kThreads + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kThreads) {
    uint64_t h;
    int sg;
    rng::cs_hash(seed, (uint64_t)j, mK_mask, h, sg);
    keys[j] = sg > 0 ? (int)h : ~(int)h;
    rank[j] = atomicAdd(cntK + h, 1);
  }
}
__global__ __launch_bounds__(kThreads) void cs_place_kernel(int64_t n, const int* __restrict__ off,
                                                            const int* __restrict__ keys,
                                                            const int* __restrict__ rank,
                                                            int* __restrict__ list) {
  for (int64_t j = blockIdx.x * (int64_t)kThreads + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kThreads) {
    const int key = keys[j];
    list[off[key < 0 ? ~key : key] + rank[j]] = key < 0 ? ~(int)j : (int)j;
  }
}

// bucket sizes of S_hat (more buckets than a wave's LDS counts)
__global__ __launch_bounds__(kThreads) void cs_count_kernel(int64_t n, uint64_t seed, int64_t r,
                                                            int* __restrict__ cntH) {
  for (int64_t j = blockIdx.x * (int64_t)kThreads + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kThreads) {
    uint64_t hh;
    int sh;
    rng::cs_hash_hat(seed, (uint64_t)j, (uint64_t)r, hh, sh);
    atomicAdd(cntH + hh, 1);
  }
}

// The Hessian buckets' lists in row order, without atomics on their (hot)
// cursors: wave w owns the contiguous rows [w C, (w + 1) C).  It counts its
// rows per bucket; a scan over the waves of every bucket gives each wave the
// first slot of its rows in every bucket; the wave then lists its rows in
// order, 64 at a time (a row's place among the batch's rows of its bucket
// comes from comparing buckets across the lanes).  Up to kHistLds buckets.
// 1024 waves: each has a row of counts, one per bucket, that is cleared, written, scanned
// and read again, so many buckets pay for more of them (twice as many waves below 2^21
// rows: 100000 x 8 float32 in 8192 buckets 145 -> 220 us, in 1000 79 -> 87 us, and
// 2 10^6 x 8 in 400 357 -> 353 us).
constexpr int kListWaves = 1024;

// per wave: its rows' counts per bucket (cntW row w), and the bucket sizes
// (integer sums: the order of the additions does not matter).  Four waves to a
// block (fewer where their counts would not fit in 64 KB of LDS), whose counts
// are added before they go to the global totals: every wave adding its own took
// 20 us of atomics on a few hundred addresses.
constexpr int kCountWaves = 4;
int cs_count_waves(int64_t buckets) {
  int w = kCountWaves;
  while (w > 1 && w * buckets * (int64_t)sizeof(int) > 65536) w /= 2;
  return w;
}
// the block's counts of n buckets (hist: one row of n per wave, the first the launch's
// wave w0) to the waves' rows of cntW, and totals += their sums
__device__ __forceinline__ void put_block_counts(const int* hist, int64_t n, int64_t w0, int waves,
                                                 int* __restrict__ cntW, int* __restrict__ tot) {
  const int nw = (int)min((int64_t)(blockDim.x >> 6), waves - w0);
  auto put = [&](auto waves_here) {
    constexpr int W = decltype(waves_here)::value;
#pragma unroll 4
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
      int c = 0;
#pragma unroll
      for (int q = 0; q < W; ++q) {
        const int v = hist[q * n + k];
        cntW[(w0 + q) * n + k] = v;
        c += v;
      }
      if (c) atomicAdd(tot + k, c);
    }
  };
  static_assert(kCountWaves == 4, "one form per number of waves");
  if (nw == 4) put(std::integral_constant<int, 4>{});
  if (nw == 3) put(std::integral_constant<int, 3>{});
  if (nw == 2) put(std::integral_constant<int, 2>{});
  if (nw == 1) put(std::integral_constant<int, 1>{});
}
__global__ __launch_bounds__(64 * kCountWaves) void cs_hat_count_kernel(
    int64_t n, int64_t chunk, int waves, uint64_t seed, int64_t r, int* __restrict__ cntW,
    int* __restrict__ cntH) {
  extern __shared__ int s_hist[];  // waves of the block x r
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
  int* hist = s_hist + wave * r;
  for (int k = lane; k < r; k += 64) hist[k] = 0;
  __syncthreads();
  const int64_t j0 = w * chunk, j1 = min(n, j0 + chunk);
  for (int64_t j = j0 + lane; j < j1; j += 64) {
    uint64_t hh;
    int sh;
    rng::cs_hash_hat(seed, (uint64_t)j, (uint64_t)r, hh, sh);
    atomicAdd(hist + hh, 1);
  }
  __syncthreads();
  put_block_counts(s_hist, r, w - wave, waves, cntW, cntH);
}

// per bucket: the exclusive scan of the bucket totals (written to off, with
// off[r] = their sum) and the first slot of every wave's rows (in place over
// the counts).  A block takes 16 buckets: its threads first sum the totals
// before them and 16 lanes scan its own; then 64 thread groups each sum a 64th
// of the waves' rows (a group's threads on consecutive buckets), the partial sums
// are scanned in LDS, and every group writes its rows' running starts.  What
// bounds it is the chain of a group's loads, so the groups are many and short
// (384 buckets, 1024 waves: 10.7 us with 64 buckets and 16 groups per block, 6.4 us so).  Integer
// sums: exact in any order.
constexpr int kColTile = 16;
constexpr int kColGroups = 1024 / kColTile;
__global__ __launch_bounds__(1024) void cs_colscan_kernel(int64_t r, int waves,
                                                          int* __restrict__ cntW,
                                                          const int* __restrict__ tot,
                                                          int* __restrict__ off) {
  __shared__ int part[kColGroups][kColTile];
  __shared__ int red[16];
  __shared__ int base[kColTile];
  const int c = threadIdx.x % kColTile, g = threadIdx.x / kColTile;
  const int64_t c0 = (int64_t)blockIdx.x * kColTile;
  const int64_t k = c0 + c;
  int pre = 0;
  for (int64_t e = threadIdx.x; e < c0; e += 1024) pre += tot[e];
  for (int m = 32; m > 0; m >>= 1) pre += __shfl_xor(pre, m, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = pre;
  // (both walks over the waves' rows load 16 counts at a time, so that their
  // loads are in flight together instead of one after another)
  constexpr int kB = 16;
  const int per = (waves + kColGroups - 1) / kColGroups;
  const int w0 = min(waves, g * per), w1 = min(waves, w0 + per);
  int t = 0;
  if (k < r) {
    int w = w0;
    for (; w + kB <= w1; w += kB) {
      int v[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) v[u] = cntW[(int64_t)(w + u) * r + k];
#pragma unroll
      for (int u = 0; u < kB; ++u) t += v[u];
    }
    for (; w < w1; ++w) t += cntW[(int64_t)w * r + k];
  }
  part[g][c] = t;
  __syncthreads();
  if (threadIdx.x < kColTile) {
    int p0 = 0;
    for (int h = 0; h < 16; ++h) p0 += red[h];
    const int own = k < r ? tot[k] : 0;
    int incl = own;
    for (int m = 1; m < kColTile; m <<= 1) {
      const int v = __shfl_up(incl, m, kColTile);
      if (c >= m) incl += v;
    }
    base[c] = p0 + incl - own;
    if (k < r) off[k] = p0 + incl - own;
    if (k == r - 1) off[r] = p0 + incl;
  }
  __syncthreads();
  if (k < r) {
    int run = base[c];
    for (int h = 0; h < g; ++h) run += part[h][c];
    int w = w0;
    for (; w + kB <= w1; w += kB) {
      int v[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) v[u] = cntW[(int64_t)(w + u) * r + k];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        cntW[(int64_t)(w + u) * r + k] = run;
        run += v[u];
      }
    }
    for (; w < w1; ++w) {
      const int n = cntW[(int64_t)w * r + k];
      cntW[(int64_t)w * r + k] = run;
      run += n;
    }
  }
}

// The largest level's lists by a stable two-pass counting sort of the rows
// on their bucket h(j) (low digit, then high digit of at most kDigitBits
// bits each), each pass in the per-wave scheme above: every wave owns a
// contiguous range of positions, counts it per digit, a scan over the waves
// of every digit gives it its first slots, and it writes its positions in
// order.  The result lists every bucket's rows in increasing row order with
// no atomic slot claims.
constexpr int kDigitBits = 11;
constexpr int kDigits = 1 << kDigitBits;
// From here the sort is faster than placing the rows by rank and sorting each list: float64
// x 64 in five levels (rank, sort) 2^17 rows 140, 161 us; 2^20 614, 627; 2^21 1171, 1168;
// 2^22 2423, 2327; float32 x 8 100, 124; 273, 288; 498, 488; 999, 893.
constexpr int64_t kRadixRows = int64_t(1) << 21;

// the rank of this lane among the batch's lanes with the same digit, and
// whether it is the last of them (one ballot per digit bit)
__device__ __forceinline__ void digit_rank(int dg, bool valid, int bits, int& before, bool& last) {
  const int lane = threadIdx.x & 63;
  uint64_t same = __ballot(valid);
  for (int b = 0; b < bits; ++b) {
    const uint64_t ones = __ballot((dg >> b) & 1);
    same &= ((dg >> b) & 1) ? ones : ~ones;
  }
  const uint64_t below = (uint64_t(1) << lane) - 1;
  before = __popcll(same & below);
  last = (same & ~below & ~(uint64_t(1) << lane)) == 0;
}

// PASS 0 draws the rows' buckets (digit = low bits); PASS 1 reads the first
// pass's keys (digit = the bits above shift)
template <int PASS>
__global__ __launch_bounds__(64 * kCountWaves) void cs_digit_count_kernel(
    int64_t n, int64_t chunk, int waves, uint64_t seed, uint64_t mK_mask, int shift, int bits,
    const int* __restrict__ keys, int* __restrict__ cntW, int* __restrict__ tot) {
  extern __shared__ int s_hist[];  // waves of the block x nd
  const int nd = 1 << bits;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
  int* hist = s_hist + wave * nd;
  for (int k = lane; k < nd; k += 64) hist[k] = 0;
  __syncthreads();
  const int64_t j0 = w * chunk, j1 = min(n, j0 + chunk);
  if constexpr (PASS == 0) {
    for (int64_t j = j0 + lane; j < j1; j += 64) {
      uint64_t h;
      int sg;
      rng::cs_hash(seed, (uint64_t)j, mK_mask, h, sg);
      atomicAdd(hist + (((int)h >> shift) & (nd - 1)), 1);
    }
  } else {
    // four rows per thread per round, their loads in flight together
    for (int64_t jb = j0 + lane; jb < j1; jb += 256) {
      int key[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) key[u] = jb + 64 * u < j1 ? keys[jb + 64 * u] : -1;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (key[u] >= 0) atomicAdd(hist + ((key[u] >> shift) & (nd - 1)), 1);
    }
  }
  __syncthreads();
  put_block_counts(s_hist, nd, w - wave, waves, cntW, tot);
}

// PASS 0: writes (bucket, entry) of every row in low-digit order; PASS 1:
// moves them into high-digit order, writing the entries (the lists) and the
// buckets in the final order
template <int PASS>
__global__ __launch_bounds__(64) void cs_digit_fill_kernel(int64_t n, int64_t chunk, uint64_t seed,
                                                           uint64_t mK_mask, int shift, int bits,
                                                           const int* __restrict__ offW,
                                                           const int* __restrict__ keys_in,
                                                           const int* __restrict__ vals_in,
                                                           int* __restrict__ keys_out,
                                                           int* __restrict__ vals_out) {
  __shared__ int cur[kDigits];
  const int lane = threadIdx.x;
  const int nd = 1 << bits;
  for (int k = lane; k < nd; k += 64) cur[k] = offW[(int64_t)blockIdx.x * nd + k];
  __syncthreads();
  const int64_t j0 = (int64_t)blockIdx.x * chunk, j1 = min(n, j0 + chunk);
  for (int64_t jb = j0; jb < j1; jb += 64) {
    const int64_t j = jb + lane;
    const bool valid = j < j1;
    int key = 0, val = 0;
    if (valid) {
      if constexpr (PASS == 0) {
        uint64_t h;
        int sg;
        rng::cs_hash(seed, (uint64_t)j, mK_mask, h, sg);
        key = (int)h;
        val = sg > 0 ? (int)j : ~(int)j;
      } else {
        key = keys_in[j];
        val = vals_in[j];
      }
    }
    const int dg = (key >> shift) & (nd - 1);
    int before;
    bool last;
    digit_rank(dg, valid, bits, before, last);
    if (valid) {
      // every lane reads its cursor before any lane writes one (one wave)
      const int slot = cur[dg] + before;
      keys_out[slot] = key;
      vals_out[slot] = val;
      if (last) cur[dg] = slot + 1;
    }
  }
}

// bucket starts from the bucket-sorted keys: position i starts every bucket
// in (key[i-1], key[i]], and the buckets past the last key start at n
__global__ void cs_starts_kernel(int64_t n, int64_t nb, const int* __restrict__ keys,
                                 int* __restrict__ off) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t lo = i == 0 ? 0 : (int64_t)keys[i - 1] + 1;
    const int64_t hi = i == n ? nb : (int64_t)keys[i];
    for (int64_t k = lo; k <= hi; ++k) off[k] = (int)i;
  }
}

__global__ __launch_bounds__(64) void cs_hat_fill_kernel(int64_t n, int64_t chunk, uint64_t seed,
                                                         int64_t r, int bits,
                                                         const int* __restrict__ offW,
                                                         int* __restrict__ listH) {
  extern __shared__ int cur[];  // r cursors
  const int lane = threadIdx.x;
  for (int k = lane; k < r; k += 64) cur[k] = offW[(int64_t)blockIdx.x * r + k];
  __syncthreads();
  const int64_t j0 = (int64_t)blockIdx.x * chunk, j1 = min(n, j0 + chunk);
  for (int64_t jb = j0; jb < j1; jb += 64) {
    const int64_t j = jb + lane;
    int hh = -1, sh = 1;
    if (j < j1) {
      uint64_t b;
      rng::cs_hash_hat(seed, (uint64_t)j, (uint64_t)r, b, sh);
      hh = (int)b;
    }
    // lanes with the same bucket: one ballot per bucket bit, and the valid lanes
    uint64_t same = __ballot(hh >= 0);
    for (int b = 0; b < bits; ++b) {
      const uint64_t ones = __ballot((hh >> b) & 1);
      same &= ((hh >> b) & 1) ? ones : ~ones;
    }
    const uint64_t below = (uint64_t(1) << lane) - 1;
    const int before = __popcll(same & below);
    const int after = __popcll(same & ~below & ~(uint64_t(1) << lane));
    if (hh >= 0) {
      // every lane reads its cursor before any lane writes one (one wave:
      // its LDS accesses take effect in program order)
      const int slot = cur[hh] + before;
      listH[slot] = sh > 0 ? (int)j : ~(int)j;
      if (after == 0) cur[hh] = slot + 1;  // the batch's last row in this bucket
    }
  }
}

// The Hessian lists and the first (low-digit) pass of the largest level's
// counting sort in one pass over the rows: both walk the same per-wave row
// ranges, so one kernel hashes each row once for the count and once for the
// fill.  Count: per wave, its rows per Hessian bucket (cntW) and per low
// digit (cntWd), and the totals of both.
__global__ __launch_bounds__(64 * kCountWaves) void cs_lists_count_kernel(
    int64_t n, int64_t chunk, int waves, uint64_t seed, int64_t r, uint64_t mK_mask, int bits,
    int* __restrict__ cntW, int* __restrict__ cntH, int* __restrict__ cntWd,
    int* __restrict__ dtot) {
  extern __shared__ int s_hist[];  // waves of the block x r, then x nd
  const int nd = 1 << bits;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int64_t w = (int64_t)blockIdx.x * nw + wave;
  int* hist = s_hist + wave * r;
  int* s_histd = s_hist + nw * r;
  int* histd = s_histd + wave * nd;
  for (int k = lane; k < r; k += 64) hist[k] = 0;
  for (int k = lane; k < nd; k += 64) histd[k] = 0;
  __syncthreads();
  const int64_t j0 = w * chunk, j1 = min(n, j0 + chunk);
  for (int64_t j = j0 + lane; j < j1; j += 64) {
    uint64_t hh, h;
    int sh, sg;
    rng::cs_hash_hat(seed, (uint64_t)j, (uint64_t)r, hh, sh);
    rng::cs_hash(seed, (uint64_t)j, mK_mask, h, sg);
    atomicAdd(hist + hh, 1);
    atomicAdd(histd + ((int)h & (nd - 1)), 1);
  }
  __syncthreads();
  put_block_counts(s_hist, r, w - wave, waves, cntW, cntH);
  put_block_counts(s_histd, nd, w - wave, waves, cntWd, dtot);
}

// Fill: every row into its Hessian bucket's list (listH) and, by its low
// digit, its (bucket, entry) into the first pass's order (keys_out, vals_out)
__global__ __launch_bounds__(64) void cs_lists_fill_kernel(
    int64_t n, int64_t chunk, uint64_t seed, int64_t r, int hbits, const int* __restrict__ offW,
    int* __restrict__ listH, uint64_t mK_mask, int bits, const int* __restrict__ offWd,
    int* __restrict__ keys_out, int* __restrict__ vals_out) {
  __shared__ int cur[kHistLds];
  __shared__ int curd[kDigits];
  const int lane = threadIdx.x;
  const int nd = 1 << bits;
  for (int k = lane; k < r; k += 64) cur[k] = offW[(int64_t)blockIdx.x * r + k];
  for (int k = lane; k < nd; k += 64) curd[k] = offWd[(int64_t)blockIdx.x * nd + k];
  __syncthreads();
  const int64_t j0 = (int64_t)blockIdx.x * chunk, j1 = min(n, j0 + chunk);
  for (int64_t jb = j0; jb < j1; jb += 64) {
    const int64_t j = jb + lane;
    const bool valid = j < j1;
    int hh = 0, sh = 1, key = 0, sg = 1;
    if (valid) {
      uint64_t b, h;
      rng::cs_hash_hat(seed, (uint64_t)j, (uint64_t)r, b, sh);
      rng::cs_hash(seed, (uint64_t)j, mK_mask, h, sg);
      hh = (int)b;
      key = (int)h;
    }
    int before, beforeD;
    bool last, lastD;
    digit_rank(hh, valid, hbits, before, last);
    const int dg = key & (nd - 1);
    digit_rank(dg, valid, bits, beforeD, lastD);
    if (valid) {
      // every lane reads its cursors before any lane writes one (one wave)
      const int slot = cur[hh] + before;
      const int slotD = curd[dg] + beforeD;
      listH[slot] = sh > 0 ? (int)j : ~(int)j;
      keys_out[slotD] = key;
      vals_out[slotD] = sg > 0 ? (int)j : ~(int)j;
      if (last) cur[hh] = slot + 1;
      if (lastD) curd[dg] = slotD + 1;
    }
  }
}

// exclusive scan of n ints in three steps: per-block scans of kScanTile
// elements with block totals, one block scanning the totals, then the carry
constexpr int kScanTile = kThreads * 8;

__global__ __launch_bounds__(kThreads) void scan_tiles_kernel(const int* __restrict__ in,
                                                              int* __restrict__ out, int64_t n,
                                                              int* __restrict__ totals) {
  __shared__ int s_w[kWaves];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
  int v[8];
  int run = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    v[q] = base + q < n ? in[base + q] : 0;
    const int t = v[q];
    v[q] = run;  // exclusive inside the thread
    run += t;
  }
  // inclusive scan of the thread totals across the block
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_w[wave] = x;
  __syncthreads();
  int wave_off = 0;
  for (int w = 0; w < wave; ++w) wave_off += s_w[w];
  const int excl = x - run + wave_off;
#pragma unroll
  for (int q = 0; q < 8; ++q)
    if (base + q < n) out[base + q] = v[q] + excl;
  if (threadIdx.x == kThreads - 1) totals[blockIdx.x] = excl + run;
}

// one block: exclusive scan of the tile totals in place, grand total to *total
__global__ __launch_bounds__(kThreads) void scan_totals_kernel(int* __restrict__ totals, int64_t nt,
                                                               int* __restrict__ total) {
  __shared__ int s_w[kWaves];
  __shared__ int s_carry;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t b0 = 0; b0 < nt; b0 += kThreads) {
    const int64_t i = b0 + threadIdx.x;
    const int v = i < nt ? totals[i] : 0;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    int wave_off = 0;
    for (int w = 0; w < wave; ++w) wave_off += s_w[w];
    const int carry = s_carry;
    if (i < nt) totals[i] = carry + wave_off + x - v;
    __syncthreads();
    if (threadIdx.x == kThreads - 1) s_carry = carry + wave_off + x;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = s_carry;
}

__global__ void scan_carry_kernel(int* __restrict__ out, int64_t n, const int* __restrict__ totals) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] += totals[i / kScanTile];
}

// list every row in its bucket of S_hat: entry = j, or ~j when the sign is -1
__global__ __launch_bounds__(kThreads) void cs_fill_kernel(int64_t n, uint64_t seed, int64_t r,
                                                           int* __restrict__ curH,
                                                           int* __restrict__ listH) {
  for (int64_t j = blockIdx.x * (int64_t)kThreads + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kThreads) {
    uint64_t hh;
    int sh;
    rng::cs_hash_hat(seed, (uint64_t)j, (uint64_t)r, hh, sh);
    listH[atomicAdd(curH + hh, 1)] = sh > 0 ? (int)j : ~(int)j;
  }
}

// These claim slots with atomics, so the order of a bucket's rows varies
// from run to run, and with it the rounding of the bucket's sum.  Sorting
// every bucket's entries by row index afterwards makes the lists, and every
// sum over them, the same on every run.  An entry is j or ~j (negative sign).
__device__ __forceinline__ int cs_row(int e) { return e < 0 ? ~e : e; }

// one thread per bucket: insertion sort in place (the largest level's buckets
// hold about N / m_K rows, two on average)
__global__ void cs_sort_small_kernel(int64_t nb, const int* __restrict__ off, int* __restrict__ list) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nb;
       k += (int64_t)gridDim.x * blockDim.x) {
    const int a = off[k], b = off[k + 1];
    for (int i = a + 1; i < b; ++i) {
      const int e = list[i];
      const int key = cs_row(e);
      int p = i - 1;
      while (p >= a && cs_row(list[p]) > key) {
        list[p + 1] = list[p];
        --p;
      }
      list[p + 1] = e;
    }
  }
}

// One block per bucket: a sorting network whose compare-exchanges all put the
// smaller key at the lower index (each merge first compares mirrored
// positions, then halves), so the length need not be a power of 2: missing
// positions act as +infinity and never move.  Segments up to kSortLds entries
// are sorted in LDS, longer ones in place in global memory.
constexpr int kSortLds = 16384;
constexpr int kSortThreads = 1024;

// LOCAL: v is in LDS, where a wave's accesses take effect in program order,
// so the sub-steps that stay inside one wave's 128 positions (t <= 128: the
// wave's 64 consecutive pairs) need no block barrier.
template <bool LOCAL, typename P>
__device__ __forceinline__ void cs_block_sort(P v, int len) {
  int span = 1;
  while (span < len) span <<= 1;
  for (int s = 2; s <= span; s <<= 1) {
    for (int t = s, lh = __builtin_ctz((unsigned)s) - 1; t >= 2; t >>= 1, --lh) {
      const bool sync = !LOCAL || t > 128;
      if (sync) __syncthreads();
      // first sub-step of a merge of size s: mirrored pairs; then half-cleaners
      // (pair q: block q >> lh of t positions, offset q mod t / 2 in it)
      const int half = t >> 1;
      for (int q = threadIdx.x; q < span / 2; q += kSortThreads) {
        const int r = q & (half - 1);
        const int i = ((q >> lh) << (lh + 1)) + r;
        const int l = (t == s) ? i - r + t - 1 - r : i + half;
        if (l < len) {
          const int x = v[i], y = v[l];
          if (cs_row(x) > cs_row(y)) {
            v[i] = y;
            v[l] = x;
          }
        }
      }
      if (sync) __syncthreads();
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(kSortThreads) void cs_sort_large_kernel(int64_t nb,
                                                                     const int* __restrict__ off,
                                                                     int* __restrict__ list) {
  __shared__ int tile[kSortLds];
  for (int64_t k = blockIdx.x; k < nb; k += gridDim.x) {
    const int a = off[k], len = off[k + 1] - a;
    if (len <= 1) continue;
    if (len <= kSortLds) {
      for (int i = threadIdx.x; i < len; i += kSortThreads) tile[i] = list[a + i];
      __syncthreads();
      cs_block_sort<true>(tile, len);
      for (int i = threadIdx.x; i < len; i += kSortThreads) list[a + i] = tile[i];
      __syncthreads();
    } else {
      cs_block_sort<false>(list + a, len);
    }
  }
}

// Rows of X read through a list are spread over lane groups: a row takes `lpr`
// lanes (a power of 2) of VEC columns each, CH such chunks per pass, and a wave
// holds 64 / lpr rows side by side, so rows narrower than a wave's 64 VEC columns
// leave no lane idle.  The 16-byte loads take any element address; where d ends
// inside a vector, the last vector is moved back to end with the row and its
// lane writes only the columns that no other lane holds.
template <typename T, int VEC>
struct ElemVec {
  typedef T type __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
};
template <typename T>
struct ElemVec<T, 1> {
  using type = T;
};
template <typename T, int VEC>
__device__ __forceinline__ void load_elems(const T* p, T (&x)[VEC]) {
  using V = typename ElemVec<T, VEC>::type;
  const V v = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  if constexpr (VEC == 1) {
    x[0] = v;
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) x[i] = v[i];
  }
}

// out row (bucket b, part p of P): sum of s(j) [x_j | y_j] over list entries
// [off[b] + p len / P, off[b] + (p + 1) len / P), len = off[b+1] - off[b].
// One wave per (bucket, part): its lane groups take every (64 / lpr)-th entry, U
// rows of each in flight, and are summed at the end.
template <typename T, int VEC, int CH>
__global__ __launch_bounds__(kThreads) void cs_gather_kernel(int64_t nb, int parts, int d, int lanes,
                                                             const T* __restrict__ X, int64_t ldx,
                                                             const T* __restrict__ Y,
                                                             const int* __restrict__ off,
                                                             const int* __restrict__ list,
                                                             T* __restrict__ out, int64_t ldo) {
  const int lane = threadIdx.x & 63;
  const int lpr = CH > 1 ? 64 : lanes;  // several chunks a pass: rows wider than a wave
  const int groups = 64 / lpr, grp = lane / lpr, l = lane & (lpr - 1);
  const int64_t nw = nb * parts;
  for (int64_t w = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6); w < nw;
       w += (int64_t)gridDim.x * kWaves) {
    const int64_t b = w / parts;
    const int p = (int)(w % parts);
    const int o0 = off[b], len = off[b + 1] - o0;
    const int e0 = o0 + (int)((int64_t)len * p / parts);
    const int e1 = o0 + (int)((int64_t)len * (p + 1) / parts);
    T* orow = out + w * ldo;
    // rows per lane group in flight: eight, but two of a row's chunks at a time
    // for rows wider than a wave, whose 2 KB runs the memory serves faster with
    // fewer of them open (2^22 x 512 float32: 5.47 ms per sketch with four, 5.37 with two)
    constexpr int U = CH > 1 ? 2 : 8;
    for (int c0 = 0; c0 < d; c0 += lpr * VEC * CH) {
      int col[CH], at[CH];
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        col[h] = c0 + (h * lpr + l) * VEC;
        at[h] = min(col[h], d - VEC);
      }
      T acc[CH][VEC];
#pragma unroll
      for (int h = 0; h < CH; ++h)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[h][v] = 0;
      // U entries per group from e; PART: those past the end are not added
      auto batch = [&](int e, auto part) {
        constexpr bool PART = decltype(part)::value;
        T x[U][CH][VEC];
        int ent[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int eu = e + u * groups + grp;
          ent[u] = list[PART ? min(eu, e1 - 1) : eu];
          const int64_t j = ent[u] < 0 ? (int64_t)~ent[u] : (int64_t)ent[u];
          const T* xr = X + j * ldx;
#pragma unroll
          for (int h = 0; h < CH; ++h) load_elems<T, VEC>(xr + at[h], x[u][h]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = !PART || e + u * groups + grp < e1;
          const T sign = ent[u] < 0 ? (T)-1 : (T)1;
#pragma unroll
          for (int h = 0; h < CH; ++h)
#pragma unroll
            for (int v = 0; v < VEC; ++v)
              acc[h][v] = fma(sign, in ? x[u][h][v] : (T)0, acc[h][v]);
        }
      };
      int e = e0;
      for (; e + U * groups <= e1; e += U * groups) batch(e, std::false_type{});
      if (e < e1) batch(e, std::true_type{});
      for (int m = lpr; m < 64; m <<= 1)
#pragma unroll
        for (int h = 0; h < CH; ++h)
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[h][v] += __shfl_xor(acc[h][v], m, 64);
      if (grp == 0) {
#pragma unroll
        for (int h = 0; h < CH; ++h)
#pragma unroll
          for (int v = 0; v < VEC; ++v)
            if (at[h] + v >= col[h]) orow[at[h] + v] = acc[h][v];
      }
    }
    // the Y column: lanes split the list, then a wave sum in lane order
    T yacc = 0;
    for (int e = e0 + lane; e < e1; e += 64) {
      const int ent = list[e];
      const int64_t j = ent < 0 ? (int64_t)~ent : (int64_t)ent;
      const T y = Y[j];
      yacc += ent < 0 ? -y : y;
    }
    for (int m = 32; m > 0; m >>= 1) yacc += __shfl_xor(yacc, m, 64);
    if (lane == 0) orow[d] = yacc;
  }
}

// Level K straight from [X|Y] together with the L levels below it (levels
// of m_K / 2, .., m_K / 2^L buckets, when the schedule has them).  One lane group
// per family of B = 2^L level-K buckets k_q = f + q mf (q < B, mf = m_K / B):
// by h(j) mod m_i, the rows of the whole family land in bucket f of level
// K - L.  The group gathers the family's rows (about 2B of them, eight loads in
// flight), keeps the B bucket sums of its columns in registers
// and writes them with their halvings: level K - l receives the B / 2^l sums
// A_{K-l}[f + q mf] = A_{K-l+1}[f + q mf] + A_{K-l+1}[f + (q + B / 2^l) mf],
// the fold fold(A)[k] = A[k] + A[k + m/2] of the smaller levels.
struct FamilyTargets {
  int64_t off[4];  // off[l]: first row (in A) of level K - l, l = 0..L
};

// Rows wider than a wave (CH > 1): at most six waves per SIMD, which has fewer of their
// runs open at once (one level of 2^20 buckets, 2.5 10^6 x 512 float32: 2548 us with the
// seven that the registers allow, 2498 with six; 1.5 10^6 x 1000 2857 and 2852).
template <typename T, int VEC, int L, int CH>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(1, CH > 1 ? 6 : 8))) void cs_gather_family_kernel(
    int64_t mf, int d, int lanes, const T* __restrict__ X, int64_t ldx, const T* __restrict__ Y,
    const int* __restrict__ off, const int* __restrict__ list, T* __restrict__ A, int64_t lda,
    FamilyTargets tg, bool a_vec) {
  constexpr int B = 1 << L;
  constexpr int U = 8 / CH;  // rows per batch: eight loads in flight
  const int lane = threadIdx.x & 63;
  const int lpr = CH > 1 ? 64 : lanes;
  const int groups = 64 / lpr, grp = lane / lpr, l = lane & (lpr - 1);
  for (int64_t f0 = ((int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6)) * groups; f0 < mf;
       f0 += (int64_t)gridDim.x * kWaves * groups) {
    // the groups past the last family repeat it without rows and without stores
    const bool live = CH > 1 || f0 + grp < mf;
    const int64_t f = live ? f0 + grp : mf - 1;
    // lane l < B of the group: the list range of bucket k_l (lpr >= 8 >= B)
    int o0 = 0, len = 0;
    if (l < B) {
      const int64_t k = f + (int64_t)l * mf;
      o0 = off[k];
      len = live ? off[k + 1] - o0 : 0;
    }
    // every lane keeps each bucket's list offset and first entry index
    int oo[B], st[B];
    int E = 0;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      oo[q] = __shfl(o0, q, lpr);
      st[q] = E;
      E += __shfl(len, q, lpr);
    }
    int Emax = E;  // of the wave's groups
    for (int m = lpr; m < 64; m <<= 1) Emax = max(Emax, __shfl_xor(Emax, m, 64));
    // bucket and list position of the family's entry e
    auto locate = [&](int e, int& qe, int& pos) {
      qe = 0;
      int oq = oo[0], sq = 0;
#pragma unroll
      for (int q = 1; q < B; ++q) {
        const int on = oo[q], sn = st[q];
        const bool past = e >= sn;
        qe = past ? q : qe;
        oq = past ? on : oq;
        sq = past ? sn : sq;
      }
      pos = oq + (e - sq);
    };
    // CH chunks of lpr VEC columns per pass: a row's chunks are loaded together
    for (int c0 = 0; c0 < d; c0 += lpr * VEC * CH) {
      int col[CH], at[CH];
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        col[h] = c0 + (h * lpr + l) * VEC;
        at[h] = min(col[h], d - VEC);
      }
      T acc[CH][B][VEC];
#pragma unroll
      for (int h = 0; h < CH; ++h)
#pragma unroll
        for (int q = 0; q < B; ++q)
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[h][q][v] = (T)0;
      for (int r0 = 0; r0 < Emax; r0 += lpr) {
        // lane l of the group holds entry r0 + l of its family and the entry's bucket
        int qe, pos;
        locate(r0 + l, qe, pos);
        const int ent = r0 + l < E ? list[pos] : 0;
        const int n = min(lpr, Emax - r0);
        for (int u0 = 0; u0 < n; u0 += U) {
          T x[U][CH][VEC];
          int qu[U];
          int neg = 0;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const bool ok = u0 + u < n && r0 + u0 + u < E;
            const int src = (u0 + u) & (lpr - 1);
            const int eu = __shfl(ent, src, lpr);
            const int qs = __shfl(qe, src, lpr);
            qu[u] = ok ? qs : -1;
            const int64_t j = eu < 0 ? (int64_t)~eu : (int64_t)eu;
            neg |= (eu < 0 ? 1 : 0) << u;
            const T* xr = X + j * ldx;
#pragma unroll
            for (int h = 0; h < CH; ++h)
#pragma unroll
              for (int v = 0; v < VEC; ++v) x[u][h][v] = (T)0;
            if (ok) {
#pragma unroll
              for (int h = 0; h < CH; ++h) load_elems<T, VEC>(xr + at[h], x[u][h]);
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < B; ++q)
#pragma unroll
              for (int h = 0; h < CH; ++h)
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                  if (qu[u] == q) acc[h][q][v] += ((neg >> u) & 1) ? -x[u][h][v] : x[u][h][v];
        }
      }
      // level K, then the halvings down to level K - L
#pragma unroll
      for (int lv = 0; lv <= L; ++lv) {
        const int nq = B >> lv;
        if (lv > 0) {
#pragma unroll
          for (int q = 0; q < (B >> 1); ++q)
            if (q < nq)
#pragma unroll
              for (int h = 0; h < CH; ++h)
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[h][q][v] += acc[h][q + nq][v];
        }
        if (!live) continue;
#pragma unroll
        for (int q = 0; q < B; ++q) {
          if (q >= nq) continue;
          T* orow = A + (tg.off[lv] + f + (int64_t)q * mf) * lda;
#pragma unroll
          for (int h = 0; h < CH; ++h) {
            if constexpr (VEC > 1) {
              if (a_vec && at[h] == col[h]) {
                typedef T V __attribute__((ext_vector_type(VEC)));
                V t;
#pragma unroll
                for (int v = 0; v < VEC; ++v) t[v] = acc[h][q][v];
                // streaming stores: the levels are not read again by this
                // pass, and keeping them out of L2 leaves it to the gathers
                __builtin_nontemporal_store(t, reinterpret_cast<V*>(orow + col[h]));
                continue;
              }
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v)
              if (at[h] + v >= col[h]) orow[at[h] + v] = acc[h][q][v];
          }
        }
      }
    }
    // the Y column: the group's lanes split the entries, then one sum per
    // bucket over the group in lane order
    T ys[B];
#pragma unroll
    for (int q = 0; q < B; ++q) ys[q] = (T)0;
    for (int e = l; e < E; e += lpr) {
      int qe, pos;
      locate(e, qe, pos);
      const int ent = list[pos];
      const int64_t j = ent < 0 ? (int64_t)~ent : (int64_t)ent;
      const T y = Y[j];
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (qe == q) ys[q] += ent < 0 ? -y : y;
    }
#pragma unroll
    for (int q = 0; q < B; ++q)
      for (int m = lpr >> 1; m > 0; m >>= 1) ys[q] += __shfl_xor(ys[q], m, 64);
#pragma unroll
    for (int lv = 0; lv <= L; ++lv) {
      const int nq = B >> lv;
      if (lv > 0) {
#pragma unroll
        for (int q = 0; q < (B >> 1); ++q)
          if (q < nq) ys[q] += ys[q + nq];
      }
      if (live && l < nq) {
        T yv = ys[0];
#pragma unroll
        for (int q = 1; q < B; ++q)
          if (l == q) yv = ys[q];
        A[(tg.off[lv] + f + (int64_t)l * mf) * lda + d] = yv;
      }
    }
  }
}

// dst[b] = sum over the parts of bucket b in part order
template <typename T>
__global__ void cs_parts_kernel(const T* __restrict__ part, int parts, int64_t nb, int cols,
                                int64_t ldp, T* __restrict__ dst, int64_t ldd) {
  const int64_t n = nb * cols;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = e / cols;
    const int c = (int)(e % cols);
    T t = 0;
    for (int q = 0; q < parts; ++q) t += part[(b * parts + q) * ldp + c];
    dst[b * ldd + c] = t;
  }
}

// dst[k][c] = sum_{q < ratio} src[k + q*m][c], k < m: rows over blocks,
// columns over threads (every access coalesced along the row)
template <typename T>
__global__ void cs_fold_kernel(const T* __restrict__ src, T* __restrict__ dst, int64_t m, int ratio,
                               int cols, int64_t ld) {
  for (int64_t k = blockIdx.x; k < m; k += gridDim.x) {
    for (int c = threadIdx.x; c < cols; c += blockDim.x) {
      T t = 0;
      for (int q = 0; q < ratio; ++q) t += src[(k + (int64_t)q * m) * ld + c];
      dst[k * ld + c] = t;
    }
  }
}

// Several levels at once by repeated halving, fold(A)[k] = A[k] + A[k + m/2]:
// work item (group g < mT, column tile) holds rows g + q mT, q < R, of the
// source level (R = m_S / mT rows, a power of 2 up to kFoldMax) in LDS and
// halves them down to one row; after the halving to s rows, the level of
// s mT rows (when the schedule has it) gets rows g + q mT, q < s.  Work
// items are dealt to the XCDs in contiguous runs, so the column tiles of one
// group (the same rows) run back to back on one XCD.  The LDS tile is sized
// for the R rows at launch: a small R leaves room for many blocks per CU,
// whose loads are then in flight together.
constexpr int kFoldMax = 512;  // source rows per group
template <typename T, int VEC>
struct FoldVec {
  using type = T __attribute__((ext_vector_type(VEC)));
};
template <typename T>
struct FoldVec<T, 1> {
  using type = T;
};
struct FoldTargets {
  int64_t off[10];  // off[lg]: first row (in A) of the level of 2^lg mT rows, or -1
};

template <typename T, int VEC>
__global__ __launch_bounds__(256) void cs_fold_tree_kernel(const T* __restrict__ src,
                                                           T* __restrict__ A, int64_t lda,
                                                           int64_t mT, int lgR, int cols, int n_ct,
                                                           int64_t xcd_q, FoldTargets tg) {
  constexpr int CT = 128 / (int)sizeof(T);  // columns per tile (128 bytes)
  constexpr int NV = CT / VEC;              // vectors per row segment
  extern __shared__ __attribute__((aligned(16))) char fold_lds[];  // R x CT values
  T* tile = reinterpret_cast<T*>(fold_lds);
  int64_t bid = blockIdx.x;
  if (xcd_q > 0 && bid < 8 * xcd_q) bid = (bid & 7) * xcd_q + (bid >> 3);
  const int ct = (int)(bid % n_ct);
  const int64_t g = bid / n_ct;
  const int c0 = ct * CT;
  const int R = 1 << lgR;
  using V = typename FoldVec<T, VEC>::type;
  // load the group's R rows of this column tile (whole vectors inside the
  // row), eight vectors per thread in flight
  constexpr int U = 8;
  for (int base = threadIdx.x; base < R * NV; base += 256 * U) {
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = base + u * 256;
      const int q = e / NV, cv = (e % NV) * VEC;
      const int col = c0 + cv;
      const T* p = src + (g + (int64_t)(e < R * NV ? q : 0) * mT) * lda + col;
      if (e < R * NV && col + VEC <= cols) {
        if constexpr (VEC == 1) {
          v[u] = __builtin_nontemporal_load(p);
        } else {
          v[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
        }
      } else {
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
          const T x = (e < R * NV && col + k < cols) ? p[k] : (T)0;
          if constexpr (VEC == 1) {
            v[u] = x;
          } else {
            v[u][k] = x;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = base + u * 256;
      if (e < R * NV) *reinterpret_cast<V*>(&tile[(e / NV) * CT + (e % NV) * VEC]) = v[u];
    }
  }
  __syncthreads();
  for (int lg = lgR - 1; lg >= 0; --lg) {
    const int sz = 1 << lg;
    const int64_t off = tg.off[lg];
    for (int e = threadIdx.x; e < sz * NV; e += 256) {
      const int q = e / NV, cv = (e % NV) * VEC;
      V a = *reinterpret_cast<const V*>(&tile[q * CT + cv]);
      const V b = *reinterpret_cast<const V*>(&tile[(q + sz) * CT + cv]);
      a = a + b;
      *reinterpret_cast<V*>(&tile[q * CT + cv]) = a;
      if (off >= 0) {
        const int col = c0 + cv;
        T* p = A + (off + g + (int64_t)q * mT) * lda + col;
        if (col + VEC <= cols) {
          if constexpr (VEC == 1) {
            __builtin_nontemporal_store(a, p);
          } else {
            __builtin_nontemporal_store(a, reinterpret_cast<V*>(p));
          }
        } else {
#pragma unroll
          for (int k = 0; k < VEC; ++k) {
            if constexpr (VEC == 1) {
              if (col + k < cols) p[k] = a;
            } else {
              if (col + k < cols) p[k] = a[k];
            }
          }
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Gaussian entries: u = (w32 + 1/2) 2^-32, z = sqrt(-2 ln u1) (cos | sin)(2 pi u2)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void box_muller8(uint64_t seed, uint64_t stream, uint64_t j,
                                            uint64_t kblk, float (&z)[8]) {
  const rng::Words w = rng::philox(j, kblk, 0, 0, seed, stream);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = (uint32_t)(w.w[q] & 0xffffffffu);
    const uint32_t hi = (uint32_t)(w.w[q] >> 32);
    const float u1 = fmaf((float)lo, 2.3283064365386963e-10f, 1.1641532182693481e-10f);
    const float u2 = fmaf((float)hi, 2.3283064365386963e-10f, 1.1641532182693481e-10f);
    const float rad = sqrtf(-2.0f * logf(u1));
    float sn, cs;
    sincosf(6.283185307179586f * u2, &sn, &cs);
    z[2 * q] = rad * cs;
    z[2 * q + 1] = rad * sn;
  }
}

// Box-Muller with the hardware transcendentals (v_log_f32 is log2, v_sin_f32
// and v_cos_f32 take revolutions): about 1e-6 relative, far below the BF16
// rounding the matrix-core path applies to G afterwards.
__device__ __forceinline__ void box_muller8_words(const uint64_t (&w)[4], float (&z)[8]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = (uint32_t)(w[q] & 0xffffffffu);
    const uint32_t hi = (uint32_t)(w[q] >> 32);
    const float u1 = fmaf((float)lo, 2.3283064365386963e-10f, 1.1641532182693481e-10f);
    const float u2 = fmaf((float)hi, 2.3283064365386963e-10f, 1.1641532182693481e-10f);
    const float rad = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));
    z[2 * q] = rad * __builtin_amdgcn_cosf(u2);
    z[2 * q + 1] = rad * __builtin_amdgcn_sinf(u2);
  }
}
__device__ __forceinline__ void box_muller8_fast(uint64_t seed, uint64_t stream, uint64_t j,
                                                 uint64_t kblk, float (&z)[8]) {
  const rng::Words w = rng::philox(j, kblk, 0, 0, seed, stream);
  box_muller8_words(w.w, z);
}

constexpr int kGT = 64;  // tile (sketch rows and columns) that the split plan counts
constexpr int kGK = 32;  // data rows per step

// The lane layouts of the FP32 and FP64 matrix-core products of 16 x 16 x 4: lane
// l holds A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator r of lane l is
// C[4 (l / 16) + r][l % 16] in FP32 and C[4 r + l / 16][l % 16] in FP64.
template <typename T>
struct GaussAcc {
  typedef T type __attribute__((ext_vector_type(4)));
};
__device__ __forceinline__ GaussAcc<float>::type mfma16(float a, float b, GaussAcc<float>::type c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ GaussAcc<double>::type mfma16(double a, double b,
                                                         GaussAcc<double>::type c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename T>
__device__ __forceinline__ int acc_row(int lane, int r) {
  return sizeof(T) == 4 ? 4 * (lane >> 4) + r : 4 * r + (lane >> 4);
}

// G [X|Y] in the data's own precision on the matrix cores: 16 NW sketch rows
// x 16 NT columns per block, one sub-range of a split's data rows, kGK rows per
// step; wave w multiplies sketch rows 16 w .. 16 w + 15 with every column
// tile, so G is drawn once per column block.  Per step and SIMD a wave's draw of G
// (one Philox block and its Box-Muller per thread, about 3400 cycles) and its
// products (NT x 8 of 64 cycles in FP64, 32 in FP32) are about equal at 100
// columns, and which of the two units bounds the kernel changes with the width;
// so the two waves of a SIMD (or the blocks of a CU) take them in opposite order:
// one draws G of the next step while the other multiplies this one.  G (as
// FP32, the type that it is drawn in) and [X|Y] are double-buffered in LDS, the
// rows of X copied straight into it a dword per lane (any alignment), one
// barrier per step.  Row strides of an odd number of 16-value groups keep the
// four k of an operand read in distinct banks.  YV: Y's column is formed on the VALU
// from the operand of G that a lane holds anyway (one multiply-add per four rows), else
// it is a column of the tiles; it would take a tile of its own wherever d is a multiple
// of 16.  The two units add up more than they overlap (2^17 x 64 FP64, 1024 rows, with
// that tile: the matrix cores busy 48% of 612 us, about a third for the draw), so what
// either does not do is gained: FP64 2^17 x 64 945 -> 852 us, 2^20 x 16 1210 -> 1057,
// 16384 x 256 1468 -> 1349; FP32 670 -> 600, 1020 -> 940, 773 -> 756.
// Measured (S of 16 d rows and S_hat of 6 d; 64 x 64 tiles of VALU products,
// G drawn again per 64 columns, before): FP64 2^17 x 64 2.70 -> 0.99 ms, 65536 x 128
// 3.63 -> 1.48 ms, 16384 x 32 1.68 -> 0.10 ms; FP32 the same shapes 2.04 -> 0.69,
// 2.42 -> 0.85, 1.42 -> 0.09 ms.
template <typename T, int NT, int NW, bool YV>
__global__ __launch_bounds__(64 * NW) void gauss_kernel(int64_t N, int d, const T* __restrict__ X,
                                                        int64_t ldx, const T* __restrict__ Y,
                                                        uint64_t seed, uint64_t stream, int64_t m,
                                                        int splits, int sub, int64_t per,
                                                        int64_t sub_per, T* __restrict__ part,
                                                        int64_t ldp) {
  constexpr int MT = 16 * NW;
  constexpr int GS = MT + 16;        // row stride of the G tile
  constexpr int WS = 16 * (NT | 1);  // row stride of the [X|Y] tile
  constexpr int TW = sizeof(T) / 4;  // dwords per value
  static_assert(MT / 8 * kGK == 64 * NW, "one Philox block per thread per step");
  __shared__ __attribute__((aligned(16))) float Gs[2][kGK * GS];
  __shared__ __attribute__((aligned(16))) T Ws[2][kGK * WS];
  __shared__ T Ys[2][YV ? kGK : 1];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t k0 = (int64_t)blockIdx.x * MT;  // sketch rows
  const int c0 = blockIdx.y * 16 * NT;          // columns of [X|Y]
  const int nx = min(16 * NT, d - c0);          // columns of X in this block (can be 0)
  const int yc = d - c0;                        // Y's column in the tile
  const bool has_y = YV ? yc <= 16 * NT : yc < 16 * NT;
  const int split = blockIdx.z / sub, q = blockIdx.z % sub;
  const int64_t s_end = min(N, (split + 1) * per);
  const int64_t j_begin = min(split * per + q * sub_per, s_end);
  const int64_t j_end = min(s_end, j_begin + sub_per);
  const int steps = (int)ceil_div(j_end - j_begin, (int64_t)kGK);
  // columns past [X|Y] stay zero, and so do the rows past the range
  for (int e = t; e < 2 * kGK * WS; e += 64 * NW) Ws[0][e] = (T)0;
  if (YV && t < 2 * kGK) Ys[0][t] = (T)0;
  __syncthreads();

  const int kb = t % (MT / 8), jj = t / (MT / 8);  // this thread's Philox block of a step
  const bool draws = k0 + 8 * kb < m;
  auto draw = [&](int s) {
    if (!draws) return;  // rows past m: their products are never stored
    const int64_t j = j_begin + (int64_t)s * kGK + jj;
    float z[8];
    box_muller8(seed, stream, (uint64_t)j, (uint64_t)((k0 >> 3) + kb), z);
    const bool live = j < j_end;
    GaussAcc<float>::type lo, hi;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = live ? z[i] : 0.0f;
      hi[i] = live ? z[4 + i] : 0.0f;
    }
    float* g = &Gs[s & 1][jj * GS + 8 * kb];
    *reinterpret_cast<GaussAcc<float>::type*>(g) = lo;
    *reinterpret_cast<GaussAcc<float>::type*>(g + 4) = hi;
  };
  auto copy = [&](int s) {
    const int64_t j0 = j_begin + (int64_t)s * kGK;
    T* Wb = Ws[s & 1];
#pragma unroll
    for (int i = 0; i < kGK / NW; ++i) {
      const int k = wave + NW * i;
      if (j0 + k < j_end) {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(X + (j0 + k) * ldx + c0);
        for (int w = 0; w < nx * TW; w += 64)
          if (w + lane < nx * TW)
            __builtin_amdgcn_global_load_lds(
                (const SLSE_GLOBAL void*)(src + w + lane),
                (__attribute__((address_space(3))) void*)(reinterpret_cast<uint32_t*>(Wb + k * WS) + w),
                4, 0, 0);
      } else {  // the last step's rows past the range
        for (int c = lane; c < nx; c += 64) Wb[k * WS + c] = (T)0;
      }
    }
  };

  typename GaussAcc<T>::type acc[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[u][r] = (T)0;
  T acc_y = 0;  // sketch row lane % 16, the rows k with k % 4 = lane / 16
  const bool mine = k0 + 16 * wave < m;
  auto multiply = [&](int s) {
    if (!mine) return;
    const float* Gb = &Gs[s & 1][16 * wave + (lane & 15)];
    const T* Wb = &Ws[s & 1][lane & 15];
    T yv[YV ? kGK / 4 : 1];
    if constexpr (YV) {
#pragma unroll
      for (int ks = 0; ks < kGK; ks += 4) yv[ks / 4] = Ys[s & 1][ks + (lane >> 4)];
    }
#pragma unroll(YV ? kGK / 4 : 2)
    for (int ks = 0; ks < kGK; ks += 4) {
      const int k = ks + (lane >> 4);
      const T a = (T)Gb[k * GS];
      if constexpr (YV) acc_y = fma(a, yv[ks / 4], acc_y);
#pragma unroll
      for (int u = 0; u < NT; ++u) acc[u] = mfma16(a, Wb[k * WS + 16 * u], acc[u]);
    }
  };

  const bool draws_first = NW > 4 ? wave < NW / 2 : (blockIdx.x + blockIdx.z) & 1;
  const bool y_thread = has_y && t < kGK;
  if (steps > 0) {
    copy(0);
    draw(0);
    if (y_thread) (YV ? Ys[0][t] : Ws[0][t * WS + yc]) = j_begin + t < j_end ? Y[j_begin + t] : (T)0;
  }
  for (int s = 0; s < steps; ++s) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this step's rows of X are in LDS
    __syncthreads();
    const bool more = s + 1 < steps;
    T y = 0;
    if (more) {
      const int64_t j = j_begin + (int64_t)(s + 1) * kGK + t;
      if (y_thread && j < j_end) y = Y[j];
      copy(s + 1);
    }
    if (more && draws_first) draw(s + 1);
    multiply(s);
    if (more && !draws_first) draw(s + 1);
    if (more && y_thread) (YV ? Ys[(s + 1) & 1][t] : Ws[(s + 1) & 1][t * WS + yc]) = y;
  }
  if (!mine) return;
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t k = k0 + 16 * wave + acc_row<T>(lane, r);
      const int col = c0 + 16 * u + (lane & 15);
      if (k < m && col < d + !YV) part[((int64_t)blockIdx.z * m + k) * ldp + col] = acc[u][r];
    }
  if (!YV || !has_y) return;
  acc_y += wave_xor(acc_y, 16);
  acc_y += wave_xor(acc_y, 32);
  const int64_t k = k0 + 16 * wave + lane;
  if (lane < 16 && k < m) part[((int64_t)blockIdx.z * m + k) * ldp + d] = acc_y;
}

template <typename T, typename Acc>
__global__ void gauss_reduce_kernel(const Acc* __restrict__ part, int splits, int64_t m, int cols,
                                    int64_t ldp, T* __restrict__ A, int64_t lda) {
  const int64_t n = m * cols;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = e / cols;
    const int c = (int)(e % cols);
    Acc t = 0;
    for (int s = 0; s < splits; ++s) t += part[((int64_t)s * m + k) * ldp + c];
    A[k * lda + c] = (T)t;
  }
}

// ---------------------------------------------------------------------------
// Gaussian sketch on the matrix cores: G and [X|Y] rounded to BF16 (nearest
// even), products accumulated in FP32 by v_mfma_f32_16x16x32_bf16.  A block
// computes kMT sketch rows x kNT columns over one split of the data rows, in
// steps of kKT data rows.  [X|Y] is converted to BF16 once, by a stage pass,
// into tiles laid out column by column (every lane reads its 8 consecutive k
// as one 16-byte load).
//
// The generation of G (Philox4x64-10 and Box-Muller, about 350 VALU
// instructions per 8 entries) is the largest cost, so the waves specialise:
// on every SIMD one wave generates G and one runs the MFMAs.  A wave issues
// in order, so a wave that did both would leave the matrix core idle while it
// generates and the VALU idle while it multiplies; with one job per wave the
// SIMD issues the MFMAs of some waves between the VALU instructions of the
// others.  During step s the generator waves write the G tile of step s + 1
// into the second of two LDS buffers while the MFMA waves multiply the tiles
// of step s and copy the [X|Y] tile of step s + 1 into the second [X|Y]
// buffer (global_load_lds: straight into LDS, no registers); one barrier per
// step swaps the buffers.  The LDS tiles are unpadded: the 16-byte chunk q of
// row c sits at chunk q ^ (c % 8) of that row, so the lanes that read one
// chunk of consecutive rows hit 8 distinct 16-byte slots of every 128-byte
// line (no bank conflicts), and a wave-wide copy still fills 1 KB of LDS in
// order (each lane picks the source chunk of its slot).  Every block of
// columns generates G again, so one block covers every column of [X|Y] when
// d < kNT.
// Lane layout of v_mfma_f32_16x16x32_bf16 (pinned by the element-wise parity
// tests): lane l holds A[l%16][8(l/16)+j] and B[8(l/16)+j][l%16], j < 8;
// accumulator r of lane l is C[4(l/16)+r][l%16].
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// 16 RT sketch rows x 64 CT columns per block (every column of a d <= 575 problem
// in one block, so G is generated once), 64 data rows per step.  Eight
// waves, two per SIMD: 4 MFMA waves, each all RT 16-row tiles x CT
// 16-column tiles of v_mfma_f32_16x16x32_bf16 (36 to 40 accumulators of four
// registers at the widest; every [X|Y] element is read from LDS by one wave only), and 4
// generator waves, RT / 2 Philox blocks per thread per step, two at a time with their rounds
// interleaved (two independent chains keep one wave's VALU issue busy).
// The blocks are as wide as [X|Y] needs: with 576 columns for every d the products of
// tiles past [X|Y] and the LDS that they fill took 5.32 ms for 2 x 1536 rows of
// 2^20 x 256 (4.42 now), 1.41 ms for 2 x 384 rows of 2^20 x 64 (1.00 now).
constexpr int kMT = 64;             // sketch rows that the split plan counts per block
constexpr int kNT = 576;            // columns per column block
constexpr int kKT = 64;             // data rows per step: 8 chunks of 8 per LDS row
constexpr int kMW = 4;              // MFMA waves: 4 column quarters of all 64 rows
constexpr int kGW = 4;              // generator waves
constexpr int kGThreads = 64 * (kMW + kGW);
constexpr int kGroupStep = 64 * kGW / kKT;  // row groups of 8 that the generator waves fill at once

// FP32 -> BF16, round to nearest even: gfx950 converts two values per
// instruction (v_cvt_pk_bf16_f32), which the compiler forms from adjacent
// conversions
__device__ __forceinline__ __bf16 to_bf16_rne(float f) { return (__bf16)f; }

// element offset of (row, k) in an unpadded swizzled LDS tile of kKT columns
__device__ __forceinline__ int swz(int row, int k) {
  return row * kKT + ((((k >> 3) ^ row) & 7) << 3) + (k & 7);
}

// [X|Y] in BF16 (nearest even), cut into tiles of kKT data rows x kNT
// columns stored column by column (tile[c][k]), tiles ordered by column block
// then data-row chunk, so that every block copies its tiles with 16-byte
// loads instead of converting and transposing [X|Y] again.  Rows past N and
// columns past d are zeros.
constexpr int kStageThreads = 256;
// columns held by the tiles of column block cb: whole 32-column MFMA tiles up
// to the last one with a column of [X|Y] (cols = d + 1)
__host__ __device__ inline int gauss_tile_cols(int cols, int cb) {
  const int left = (int)round_up(cols, 32) - cb * kNT;
  return left < kNT ? left : kNT;
}
__global__ __launch_bounds__(kStageThreads) void gauss_stage_kernel(
    int64_t N, int d, const float* __restrict__ X, int64_t ldx, const float* __restrict__ Y,
    int64_t nchunks, __bf16* __restrict__ tiles) {
  const int64_t chunk = blockIdx.x;
  const int cb = blockIdx.y;
  const int64_t j0 = chunk * kKT;
  const int wc = gauss_tile_cols(d + 1, cb);
  __bf16* t = tiles + (int64_t)cb * nchunks * (kNT * kKT) + chunk * (wc * kKT);
  // FP32 rows on 16-byte boundaries: four columns per load
  const bool vec4 = (reinterpret_cast<uintptr_t>(X) % 16) == 0 && ldx % 4 == 0;
  // item (4 columns from 4 c4, 8 data rows from 8 q): eight row loads, four
  // 16-byte stores (the 8 k values of each column); consecutive threads take
  // the row groups of one column group, so that each store instruction
  // fills whole 128-byte column segments of the tile
  const int ncg = wc / 4;
  constexpr int NQG = kKT / 8;
  for (int e = threadIdx.x; e < ncg * NQG; e += kStageThreads) {
    const int q = e % NQG, c4 = e / NQG;
    const int col = cb * kNT + 4 * c4;
    float v[8][4];
    const int64_t jq = j0 + 8 * q;
    if (vec4 && col + 4 <= d && jq + 8 <= N) {
      // the common case: eight whole 16-byte loads, all in flight at once
      f32x4_t x[8];
#pragma unroll
      for (int r = 0; r < 8; ++r)
        x[r] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(X + (jq + r) * ldx + col));
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[r][i] = x[r][i];
    } else {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t j = jq + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = col + i;
          v[r][i] = j < N ? (c < d ? X[j * ldx + c] : (c == d ? Y[j] : 0.0f)) : 0.0f;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bf16x8_t w;
#pragma unroll
      for (int r = 0; r < 8; ++r) w[r] = to_bf16_rne(v[r][i]);
      __builtin_nontemporal_store(w, reinterpret_cast<bf16x8_t*>(t + (int64_t)(4 * c4 + i) * kKT + 8 * q));
    }
  }
}

// one step of the generator waves: RT / 2 Philox blocks of 8 sketch rows at
// data row j per thread, rounded to BF16 and written to the G tile (rows past
// the split are zeros)
template <int RT>
__device__ __forceinline__ void gauss_gen_step(uint64_t seed, uint64_t stream, int64_t k0,
                                               int64_t j, int64_t j_end, int gt, __bf16* Gb) {
  const int kb = gt / kKT, jj = gt % kKT;
  const bool live = j < j_end;
  static_assert(RT % 4 == 0 && kGroupStep * (RT / 2) == 2 * RT, "whole pairs of Philox blocks");
#pragma unroll
  for (int h = 0; h < RT / 2; h += 2) {
    // two blocks' rounds side by side: independent chains for the one
    // generator wave of a SIMD to issue back to back
    rng::PhiloxState st[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
      st[b] = rng::PhiloxState{{(uint64_t)j, (uint64_t)((k0 >> 3) + kb + (h + b) * kGroupStep), 0, 0},
                               seed,
                               stream};
#pragma unroll
    for (int r = 0; r < 10; ++r)
#pragma unroll
      for (int b = 0; b < 2; ++b) rng::philox_round(st[b], r);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int rb = kb + (h + b) * kGroupStep;  // group of 8 sketch rows
      float z[8];
      box_muller8_words(st[b].c, z);
#pragma unroll
      for (int q = 0; q < 8; ++q) Gb[swz(rb * 8 + q, jj)] = to_bf16_rne(live ? z[q] : 0.0f);
    }
  }
}

// the staged [X|Y] tile of one step copied straight into LDS by the MFMA
// waves (16 bytes per lane, placed in order from the wave's LDS base; no
// registers): slot p of row c receives the tile's chunk p ^ (c % 8)
__device__ __forceinline__ void gauss_copy_step(const __bf16* tb, int wc, __bf16* Wb, int wave,
                                                int lane) {
  const int copies = wc / 8;  // 8 rows of 128 bytes per wave-wide copy
  const int c_in = lane >> 3, p = lane & 7;
  for (int g = wave; g < copies; g += kMW) {
    const int c = 8 * g + c_in;
    const __bf16* src = tb + (int64_t)c * kKT + 8 * (p ^ c_in);
    __builtin_amdgcn_global_load_lds(
        (const SLSE_GLOBAL void*)src,
        (__attribute__((address_space(3))) void*)(reinterpret_cast<char*>(Wb) + 1024 * g), 16, 0,
        0);
  }
}

template <int CT, int RT>
__global__ __launch_bounds__(kGThreads) void gauss_mfma_kernel(int64_t N, int d,
                                                         const __bf16* __restrict__ tiles,
                                                         int64_t nchunks, uint64_t seed,
                                                         uint64_t stream, int64_t m, int splits,
                                                         float* __restrict__ part, int64_t ldp) {
  static_assert((2 * 64 * CT + 2 * 16 * RT) * kKT * 2 <= 163840,
                "two [X|Y] tiles and two G tiles fit in LDS");
  __shared__ __attribute__((aligned(1024))) __bf16 Ws[2][64 * CT * kKT];
  __shared__ __attribute__((aligned(1024))) __bf16 Gs[2][16 * RT * kKT];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t k0 = (int64_t)blockIdx.x * 16 * RT;
  const int split = blockIdx.z;
  const int cblk = blockIdx.y;
  const int c0 = cblk * kNT;
  const int64_t per = round_up(ceil_div(N, (int64_t)splits), kKT);
  const int64_t j_begin = (int64_t)split * per;
  const int64_t j_end = min(N, j_begin + per);
  const __bf16* tcol = tiles + (int64_t)cblk * nchunks * (kNT * kKT);
  const int wc = gauss_tile_cols(d + 1, cblk);  // columns of this block's tiles
  const int64_t steps = j_end > j_begin ? ceil_div(j_end - j_begin, kKT) : 0;
  const bool mfma_wave = wave < kMW;
  const int gt = threadIdx.x - 64 * kMW;  // generator thread index
  // step 0's tiles.  A split past the last data row (the rounding of the
  // split length can leave the last ones empty) runs no step but still
  // writes its zero partials; steps is the same for the whole block, so
  // every wave meets the same barriers.
  if (steps > 0) {
    if (mfma_wave) {
      gauss_copy_step(tcol + (j_begin / kKT) * (wc * kKT), wc, Ws[0], wave, lane);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
      gauss_gen_step<RT>(seed, stream, k0, j_begin + gt % kKT, j_end, gt, Gs[0]);
    }
    __syncthreads();
  }
  if (mfma_wave) {
    const int cq = wave;  // column group: CT 16-column tiles
    f32x4_t acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < CT; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][q][r] = 0.0f;
    for (int64_t s = 0; s < steps; ++s) {
      const int b = (int)(s & 1);
      if (s + 1 < steps)
        gauss_copy_step(tcol + ((j_begin + (s + 1) * kKT) / kKT) * (wc * kKT), wc, Ws[b ^ 1],
                        wave, lane);
      const __bf16* Gb = Gs[b];
      const __bf16* Wb = Ws[b];
#pragma unroll
      for (int ks = 0; ks < kKT / 32; ++ks) {
        const int kk = 32 * ks + 8 * (lane >> 4);
        bf16x8_t a[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i)
          a[i] = *reinterpret_cast<const bf16x8_t*>(&Gb[swz(i * 16 + (lane & 15), kk)]);
#pragma unroll
        for (int q = 0; q < CT; ++q) {
          // tiles past [X|Y] multiply stale LDS and are never stored (a
          // wave-uniform skip measured slower: it splits the unrolled loop)
          const int col = (cq * CT + q) * 16 + (lane & 15);
          const bf16x8_t bv = *reinterpret_cast<const bf16x8_t*>(&Wb[swz(col, kk)]);
#pragma unroll
          for (int i = 0; i < RT; ++i)
            acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], bv, acc[i][q], 0, 0, 0);
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // next [X|Y] tile is in LDS
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < CT; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t k = k0 + i * 16 + 4 * (lane >> 4) + r;
          const int t = cq * CT + q;
          const int col = c0 + t * 16 + (lane & 15);
          if (k < m && col <= d && t * 16 < wc)
            part[((int64_t)split * m + k) * ldp + col] = acc[i][q][r];
        }
  } else {
    for (int64_t s = 0; s < steps; ++s) {
      // G of step s + 1 (zeros after the last step: never read)
      const int64_t j = j_begin + (s + 1) * kKT + gt % kKT;
      gauss_gen_step<RT>(seed, stream, k0, j, j_end, gt, Gs[(s + 1) & 1]);
      __syncthreads();
    }
  }
}

// Reference for measurement: the matrix-core kernel's generation of G alone
// (Philox block -> eight Box-Muller values -> BF16) for entries k < m, j < N,
// folded into one checksum word per thread; no data is read and no product
// formed.  Its time is the floor the VALU work of the Gaussian sketch sets.
__global__ __launch_bounds__(256) void gauss_generate_kernel(uint64_t seed, uint64_t stream,
                                                             int64_t kblocks, int64_t N,
                                                             unsigned* __restrict__ sink) {
  const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  // entry e = kb N + j, walked with a carry instead of a division per entry
  int64_t kb = tid / N, j = tid % N;
  const int64_t skb = stride / N, sj = stride % N;
  unsigned acc = 0;
  while (kb < kblocks) {
    float z[8];
    box_muller8_fast(seed, stream, (uint64_t)j, (uint64_t)kb, z);
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += __builtin_bit_cast(uint16_t, to_bf16_rne(z[q]));
    kb += skb;
    j += sj;
    if (j >= N) {
      j -= N;
      ++kb;
    }
  }
  sink[tid] = acc;
}

// form 0: the entries of the VALU kernels; form 1: those of the matrix-core
// kernel (hardware transcendentals, then rounded to BF16 as its operands are)
__global__ void debug_gauss_kernel(uint64_t seed, uint64_t stream, int64_t k0, int64_t nk,
                                   int64_t j0, int64_t nj, int form, double* __restrict__ out) {
  const int64_t n = nk * nj;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t a = e / nj, b = e % nj;
    const int64_t k = k0 + a, j = j0 + b;
    float z[8];
    if (form == 1) {
      box_muller8_fast(seed, stream, (uint64_t)j, (uint64_t)(k >> 3), z);
      out[e] = (double)(float)(__bf16)z[k & 7];
    } else {
      box_muller8(seed, stream, (uint64_t)j, (uint64_t)(k >> 3), z);
      out[e] = (double)z[k & 7];
    }
  }
}

int grid1(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, 256), 8192)); }

// parts of each Hessian bucket: enough for about 6144 waves (six per SIMD keep
// the gather's random rows in flight), each of at least 64 rows.  2^20 x 64
// float64 in 384 buckets: 3 parts of 1024 rows on half of each wave's lanes 567 us,
// 16 parts with two rows side by side 98 us.
int cs_hat_parts(int64_t N, int64_t r) {
  const int64_t per = ceil_div(std::max<int64_t>(N, 1), std::max<int64_t>(r, 1));
  const int64_t want = ceil_div(6144, std::max<int64_t>(r, 1));
  return (int)std::max<int64_t>(1, std::min<int64_t>({64, want, ceil_div(per, 64)}));
}

// lanes per row of the gathers: VEC columns a lane, from 8 lanes (a family's
// buckets are looked up by the first 8 lanes of its group) to a wave
int cs_lanes(int d, int vec) {
  int lpr = 8;
  while (lpr < 64 && lpr * vec < d) lpr *= 2;
  return lpr;
}

__global__ void copy_i32_kernel(const int* __restrict__ src, int* __restrict__ dst, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

void copy_i32(const int* src, int* dst, int64_t n, hipStream_t s) {
  copy_i32_kernel<<<grid1(n), 256, 0, s>>>(src, dst, n);
  SLSE_LAUNCH_CHECK();
}

// Scratch of the bucket lists, carved from CountSketchArgs::scratch.
struct CsScratch {
  int *cntK, *offK, *listK, *cntH, *offH, *listH, *totals;
  int* cntW;   // per (wave, Hessian bucket) counts, then first slots (row-order fills)
  int* cntWd;  // the same per (wave, digit) for the counting sort
  int waves;
  int64_t chunk;
  bool radix;                    // the largest level's lists by the counting sort
  int *keysA, *valsA, *keysB;    // its passes' buckets and entries (keysA, valsA: or the rows'
                                 // buckets and arrival numbers)
  int *dtot, *doff;              // per-digit totals and their scan
  void* partH;
  size_t bytes;
};

CsScratch cs_scratch(const CountSketchArgs& a) {
  const int64_t mK = a.m[a.K - 1];
  const int parts = cs_hat_parts(a.N, a.r);
  const int64_t ntiles = ceil_div(std::max<int64_t>({mK, a.r, 1}), (int64_t)kScanTile);
  const size_t es = dtype_size(a.t);
  char* p = static_cast<char*>(a.scratch);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* q = p ? p + o : nullptr;
    o += (size_t)round_up((int64_t)bytes, 256);
    return q;
  };
  CsScratch c;
  c.cntK = reinterpret_cast<int*>(take(sizeof(int) * mK));
  c.offK = reinterpret_cast<int*>(take(sizeof(int) * (mK + 1)));
  c.listK = reinterpret_cast<int*>(take(sizeof(int) * a.N));
  c.cntH = reinterpret_cast<int*>(take(sizeof(int) * a.r));
  c.offH = reinterpret_cast<int*>(take(sizeof(int) * (a.r + 1)));
  c.listH = reinterpret_cast<int*>(take(sizeof(int) * a.N));
  c.totals = reinterpret_cast<int*>(take(sizeof(int) * ntiles));
  c.partH = parts > 1 ? take(es * (size_t)a.r * parts * (a.d + 1)) : nullptr;
  // per-wave row ranges: the Hessian lists in row order when their counts fit
  // in a wave's LDS; the largest level's by the counting sort when its
  // buckets take at most two digits
  const int64_t w = std::min<int64_t>(kListWaves, ceil_div(std::max<int64_t>(a.N, 1), 64));
  c.chunk = round_up(ceil_div(std::max<int64_t>(a.N, 1), w), 64);
  c.waves = (int)ceil_div(std::max<int64_t>(a.N, 1), c.chunk);
  const bool hat_rows = a.r <= kHistLds;
  c.radix = ilog2_ceil(mK) <= 2 * kDigitBits;
  c.cntW = hat_rows ? reinterpret_cast<int*>(take(sizeof(int) * (size_t)c.waves * a.r)) : nullptr;
  c.cntWd = c.radix ? reinterpret_cast<int*>(take(sizeof(int) * (size_t)c.waves * kDigits)) : nullptr;
  c.keysA = reinterpret_cast<int*>(take(sizeof(int) * a.N));
  c.valsA = reinterpret_cast<int*>(take(sizeof(int) * a.N));
  c.keysB = c.dtot = c.doff = nullptr;
  if (c.radix) {
    c.keysB = reinterpret_cast<int*>(take(sizeof(int) * a.N));
    c.dtot = reinterpret_cast<int*>(take(sizeof(int) * (kDigits + 1)));
    c.doff = reinterpret_cast<int*>(take(sizeof(int) * (kDigits + 1)));
  }
  c.bytes = o;
  return c;
}

void scan_exclusive(const int* in, int* out, int64_t n, int* totals, hipStream_t s) {
  const int64_t nt = ceil_div(std::max<int64_t>(n, 1), (int64_t)kScanTile);
  scan_tiles_kernel<<<(unsigned)nt, kThreads, 0, s>>>(in, out, n, totals);
  scan_totals_kernel<<<1, kThreads, 0, s>>>(totals, nt, out + n);
  scan_carry_kernel<<<(unsigned)ceil_div(std::max<int64_t>(n, 1), 256), 256, 0, s>>>(out, n, totals);
  SLSE_LAUNCH_CHECK();
}

template <typename T>
void gather(int64_t nb, int parts, const CountSketchArgs& a, const int* off, const int* list, T* out,
            int64_t ldo, hipStream_t s) {
  const int64_t waves = nb * parts;
  const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(waves, kWaves), 65536));
  const T* X = static_cast<const T*>(a.X);
  const T* Y = static_cast<const T*>(a.Y);
  constexpr int V = 16 / sizeof(T);
  const int lpr = cs_lanes(a.d, a.d >= V ? V : 1);
  if (a.d > 64 * V)  // rows wider than one chunk: two chunks of a row per pass
    cs_gather_kernel<T, V, 2><<<blocks, kThreads, 0, s>>>(nb, parts, a.d, lpr, X, a.ldx, Y, off, list, out, ldo);
  else if (a.d >= V)
    cs_gather_kernel<T, V, 1><<<blocks, kThreads, 0, s>>>(nb, parts, a.d, lpr, X, a.ldx, Y, off, list, out, ldo);
  else
    cs_gather_kernel<T, 1, 1><<<blocks, kThreads, 0, s>>>(nb, parts, a.d, lpr, X, a.ldx, Y, off, list, out, ldo);
  SLSE_LAUNCH_CHECK();
}

// Level K (at row offK of A) and the L levels below it, one wave per family.
template <typename T>
void gather_family(int L, const CountSketchArgs& a, const int* off, const int* list, T* A,
                   int64_t offK, hipStream_t s) {
  const int64_t mK = a.m[a.K - 1];
  const int64_t mf = mK >> L;
  FamilyTargets tg;
  int64_t o = offK;
  for (int l = 0; l < 4; ++l) tg.off[l] = -1;
  for (int l = 0; l <= L; ++l) {
    tg.off[l] = o;
    if (l < L) o -= a.m[a.K - 2 - l];
  }
  const T* X = static_cast<const T*>(a.X);
  const T* Y = static_cast<const T*>(a.Y);
  constexpr int V = 16 / sizeof(T);
  const bool vec = a.d >= V;
  const int lpr = cs_lanes(a.d, vec ? V : 1);
  const unsigned blocks = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>(ceil_div(mf, (int64_t)kWaves * (64 / lpr)), 65536));
  const bool a_vec = (reinterpret_cast<uintptr_t>(A) % 16 == 0) && ((a.lda * (int64_t)sizeof(T)) % 16 == 0);
#define SLSE_FAMILY(VV, LL, CC)                                                                 \
  cs_gather_family_kernel<T, VV, LL, CC><<<blocks, kThreads, 0, s>>>(mf, a.d, lpr, X, a.ldx, Y,    \
                                                                     off, list, A, a.lda, tg, a_vec)
  // rows wider than one chunk of 64 V columns: two chunks of a row per pass
  const bool two = a.d > 64 * V;
  if (vec && two) {
    if (L == 3) SLSE_FAMILY(V, 3, 2);
    else if (L == 2) SLSE_FAMILY(V, 2, 2);
    else if (L == 1) SLSE_FAMILY(V, 1, 2);
    else SLSE_FAMILY(V, 0, 2);
  } else if (vec) {
    if (L == 3) SLSE_FAMILY(V, 3, 1);
    else if (L == 2) SLSE_FAMILY(V, 2, 1);
    else if (L == 1) SLSE_FAMILY(V, 1, 1);
    else SLSE_FAMILY(V, 0, 1);
  } else {
    if (L == 3) SLSE_FAMILY(1, 3, 1);
    else if (L == 2) SLSE_FAMILY(1, 2, 1);
    else if (L == 1) SLSE_FAMILY(1, 1, 1);
    else SLSE_FAMILY(1, 0, 1);
  }
#undef SLSE_FAMILY
  SLSE_LAUNCH_CHECK();
}

// Levels top-1 .. 0 from level `top` (level i sits just before level i + 1
// in A, level K-1 at row offK).  Each pass folds a source level down as far as
// kFoldMax rows per group allow and writes every level on the way; a step
// between two levels wider than that falls back to the one-level fold.
template <typename T>
void fold_levels(const CountSketchArgs& a, T* A, int64_t offK, int top, hipStream_t s) {
  std::vector<int64_t> off(a.K);
  off[a.K - 1] = offK;
  for (int i = a.K - 2; i >= 0; --i) off[i] = off[i + 1] - a.m[i];
  const int cols = a.d + 1;
  constexpr int CT = 128 / (int)sizeof(T);
  const int n_ct = (int)ceil_div(cols, CT);
  const bool vec = (reinterpret_cast<uintptr_t>(A) % 16 == 0) && ((a.lda * (int64_t)sizeof(T)) % 16 == 0);
  int S = top;
  while (S > 0) {
    int Tl = S;
    while (Tl > 0 && a.m[S] / a.m[Tl - 1] <= kFoldMax) --Tl;
    if (Tl == S) {  // the next level is more than kFoldMax times smaller
      const int i = S - 1;
      cs_fold_kernel<T><<<(unsigned)std::min<int64_t>(a.m[i], 65536), 256, 0, s>>>(
          A + off[S] * a.lda, A + off[i] * a.lda, a.m[i], (int)(a.m[S] / a.m[i]), cols, a.lda);
      SLSE_LAUNCH_CHECK();
      S = i;
      continue;
    }
    const int64_t mT = a.m[Tl];
    const int lgR = ilog2_ceil(a.m[S] / mT);
    FoldTargets tg;
    for (int k = 0; k < 10; ++k) tg.off[k] = -1;
    for (int i = Tl; i < S; ++i) tg.off[ilog2_ceil(a.m[i] / mT)] = off[i];
    const int64_t blocks = mT * n_ct;
    if (blocks > 0x7fffffffLL) fail(SLSE_EUNSUPPORTED, "countsketch: too many fold work items");
    const int64_t xq = blocks / 8;
    const size_t lds = (size_t)(int64_t(1) << lgR) * CT * sizeof(T);  // at most 64 KiB
    if (vec)
      cs_fold_tree_kernel<T, 16 / sizeof(T)><<<(unsigned)blocks, 256, lds, s>>>(
          A + off[S] * a.lda, A, a.lda, mT, lgR, cols, n_ct, xq, tg);
    else
      cs_fold_tree_kernel<T, 1><<<(unsigned)blocks, 256, lds, s>>>(A + off[S] * a.lda, A, a.lda, mT,
                                                                   lgR, cols, n_ct, xq, tg);
    SLSE_LAUNCH_CHECK();
    S = Tl;
  }
}

template <typename T>
void countsketch_t(const CountSketchArgs& a, hipStream_t s) {
  if (a.N >= (int64_t(1) << 31)) fail(SLSE_EUNSUPPORTED, "countsketch: N >= 2^31 rows");
  T* A = static_cast<T*>(a.A);
  T* Ah = static_cast<T*>(a.Ahat);
  int64_t rows_A = 0;
  for (int i = 0; i < a.K; ++i) rows_A += a.m[i];
  const int64_t mK = a.m[a.K - 1];
  const CsScratch sc = cs_scratch(a);
  const unsigned rb = (unsigned)grid1(a.N);
  const uint64_t mK_mask = (uint64_t)mK - 1;
  // 1. the largest level's lists, every bucket's rows in increasing row order:
  // by the counting sort from 2^21 rows, below that placed by arrival number with
  // a sort of each list (fewer launches; the two give the same lists).
  // SLSE_CS_SORT=1 / 0 forces one of them, for measurement and tests.
  bool radix = sc.radix && a.N >= kRadixRows;
  if (const char* e = std::getenv("SLSE_CS_SORT")) radix = sc.radix && std::atoi(e) != 0;
  const bool hat_rows = a.r <= kHistLds;
  const unsigned ncs = (unsigned)ceil_div(kDigits, kColTile);
  // count kernels: waves per block, blocks and LDS for `buckets` counts per wave
  struct CountShape {
    unsigned blocks, threads;
    size_t lds;
  };
  auto count_shape = [&](int64_t buckets) {
    const int w = cs_count_waves(buckets);
    return CountShape{(unsigned)ceil_div(sc.waves, w), (unsigned)(64 * w),
                      (size_t)w * (size_t)buckets * sizeof(int)};
  };
  auto digit_pass1 = [&](int shift, int bits) {  // high digit: counts, first slots, fill
    fill_kernel<int><<<grid1(kDigits), 256, 0, s>>>(sc.dtot, 1, kDigits, kDigits);
    const CountShape cd = count_shape(int64_t(1) << bits);
    cs_digit_count_kernel<1><<<cd.blocks, cd.threads, cd.lds, s>>>(
        a.N, sc.chunk, sc.waves, a.seed, mK_mask, shift, bits, sc.keysA, sc.cntWd, sc.dtot);
    cs_colscan_kernel<<<ncs, 1024, 0, s>>>(int64_t(1) << bits, sc.waves, sc.cntWd, sc.dtot, sc.doff);
    cs_digit_fill_kernel<1><<<(unsigned)sc.waves, 64, 0, s>>>(
        a.N, sc.chunk, a.seed, mK_mask, shift, bits, sc.cntWd, sc.keysA, sc.valsA, sc.keysB, sc.listK);
  };
  if (radix && hat_rows) {
    // the Hessian lists and the low-digit pass together, then the high digit
    const int p = ilog2_ceil(mK);
    const int b0 = std::min(p, kDigitBits), b1 = p - b0;
    fill_kernel<int><<<grid1(kDigits), 256, 0, s>>>(sc.dtot, 1, kDigits, kDigits);
    fill_kernel<int><<<grid1(a.r), 256, 0, s>>>(sc.cntH, 1, a.r, a.r);
    const CountShape cl = count_shape(a.r + (int64_t(1) << b0));
    cs_lists_count_kernel<<<cl.blocks, cl.threads, cl.lds, s>>>(a.N, sc.chunk, sc.waves, a.seed, a.r,
                                                               mK_mask, b0, sc.cntW, sc.cntH,
                                                               sc.cntWd, sc.dtot);
    cs_colscan_kernel<<<ncs, 1024, 0, s>>>(int64_t(1) << b0, sc.waves, sc.cntWd, sc.dtot, sc.doff);
    cs_colscan_kernel<<<(unsigned)ceil_div(a.r, kColTile), 1024, 0, s>>>(a.r, sc.waves, sc.cntW,
                                                                        sc.cntH, sc.offH);
    cs_lists_fill_kernel<<<(unsigned)sc.waves, 64, 0, s>>>(
        a.N, sc.chunk, a.seed, a.r, ilog2_ceil(a.r), sc.cntW, sc.listH, mK_mask, b0, sc.cntWd,
        b1 ? sc.keysA : sc.keysB, b1 ? sc.valsA : sc.listK);
    if (b1) digit_pass1(b0, b1);
    cs_starts_kernel<<<grid1(a.N + 1), 256, 0, s>>>(a.N, mK, sc.keysB, sc.offK);
    SLSE_LAUNCH_CHECK();
  } else {
    if (radix) {
      const int p = ilog2_ceil(mK);
      const int b0 = std::min(p, kDigitBits), b1 = p - b0;
      fill_kernel<int><<<grid1(kDigits), 256, 0, s>>>(sc.dtot, 1, kDigits, kDigits);
      const CountShape cd = count_shape(int64_t(1) << b0);
      cs_digit_count_kernel<0><<<cd.blocks, cd.threads, cd.lds, s>>>(
          a.N, sc.chunk, sc.waves, a.seed, mK_mask, 0, b0, nullptr, sc.cntWd, sc.dtot);
      cs_colscan_kernel<<<ncs, 1024, 0, s>>>(int64_t(1) << b0, sc.waves, sc.cntWd, sc.dtot, sc.doff);
      cs_digit_fill_kernel<0><<<(unsigned)sc.waves, 64, 0, s>>>(
          a.N, sc.chunk, a.seed, mK_mask, 0, b0, sc.cntWd, nullptr, nullptr,
          b1 ? sc.keysA : sc.keysB, b1 ? sc.valsA : sc.listK);
      if (b1) digit_pass1(b0, b1);
      cs_starts_kernel<<<grid1(a.N + 1), 256, 0, s>>>(a.N, mK, sc.keysB, sc.offK);
    } else {
      fill_kernel<int><<<grid1(mK), 256, 0, s>>>(sc.cntK, 1, mK, mK);
      cs_count_rank_kernel<<<rb, kThreads, 0, s>>>(a.N, a.seed, mK_mask, sc.cntK, sc.keysA, sc.valsA);
      scan_exclusive(sc.cntK, sc.offK, mK, sc.totals, s);
      cs_place_kernel<<<rb, kThreads, 0, s>>>(a.N, sc.offK, sc.keysA, sc.valsA, sc.listK);
      cs_sort_small_kernel<<<grid1(mK), 256, 0, s>>>(mK, sc.offK, sc.listK);
    }
    SLSE_LAUNCH_CHECK();
    // 2. the Hessian buckets' lists, in row order too
    fill_kernel<int><<<grid1(a.r), 256, 0, s>>>(sc.cntH, 1, a.r, a.r);
    if (hat_rows) {
      const CountShape ch = count_shape(a.r);
      cs_hat_count_kernel<<<ch.blocks, ch.threads, ch.lds, s>>>(a.N, sc.chunk, sc.waves, a.seed, a.r,
                                                               sc.cntW, sc.cntH);
      cs_colscan_kernel<<<(unsigned)ceil_div(a.r, kColTile), 1024, 0, s>>>(a.r, sc.waves, sc.cntW,
                                                                          sc.cntH, sc.offH);
      cs_hat_fill_kernel<<<(unsigned)sc.waves, 64, sizeof(int) * (size_t)a.r, s>>>(
          a.N, sc.chunk, a.seed, a.r, ilog2_ceil(a.r), sc.cntW, sc.listH);
    } else {
      cs_count_kernel<<<rb, kThreads, 0, s>>>(a.N, a.seed, a.r, sc.cntH);
      scan_exclusive(sc.cntH, sc.offH, a.r, sc.totals, s);
      copy_i32(sc.offH, sc.cntH, a.r, s);
      cs_fill_kernel<<<rb, kThreads, 0, s>>>(a.N, a.seed, a.r, sc.cntH, sc.listH);
      cs_sort_large_kernel<<<(unsigned)std::min<int64_t>(a.r, 65535), kSortThreads, 0, s>>>(
          a.r, sc.offH, sc.listH);
    }
    SLSE_LAUNCH_CHECK();
  }
  // 3. gathers: the largest level and up to three below it straight into A,
  //    S_hat through its parts
  const int64_t offK = rows_A - mK;
  // fuse the levels below K that halve it step by step (up to three)
  int L = 0;
  while (L < 3 && L < a.K - 1 && a.m[a.K - 2 - L] == (mK >> (L + 1))) ++L;
  gather_family<T>(L, a, sc.offK, sc.listK, A, offK, s);
  const int parts = cs_hat_parts(a.N, a.r);
  if (parts == 1) {
    gather<T>(a.r, 1, a, sc.offH, sc.listH, Ah, a.ldah, s);
  } else {
    T* part = static_cast<T*>(sc.partH);
    const int64_t ldp = a.d + 1;
    gather<T>(a.r, parts, a, sc.offH, sc.listH, part, ldp, s);
    cs_parts_kernel<T><<<grid1(a.r * (a.d + 1)), 256, 0, s>>>(part, parts, a.r, a.d + 1, ldp, Ah,
                                                             a.ldah);
    SLSE_LAUNCH_CHECK();
  }
  // 4. smaller levels by folding, several levels per pass
  fold_levels<T>(a, A, offK, a.K - 1 - L, s);
}

// BF16 path scratch: the staged tiles (shared by the two sketches of one
// [X|Y]: they depend only on N and d), then, at a 256-byte boundary, the split
// partial sums
size_t gauss_partial_bytes(const GaussianArgs& a) {
  const size_t es = (a.t == SLSE_F64 && !a.bf16) ? 8 : 4;
  return (size_t)a.splits * (size_t)a.sub * (size_t)a.m * (size_t)round_up(a.d + 1, 4) * es;
}
size_t gauss_tile_bytes(const GaussianArgs& a) {
  if (!a.bf16) return 0;
  return (size_t)ceil_div(a.d + 1, kNT) * (size_t)ceil_div(std::max<int64_t>(a.N, 1), kKT) *
         (size_t)(kNT * kKT) * sizeof(__bf16);
}

void gaussian_mfma(const GaussianArgs& a, hipStream_t s) {
  const int cols = a.d + 1;
  const int64_t ldp = round_up(cols, 4);
  const int64_t nchunks = ceil_div(std::max<int64_t>(a.N, 1), kKT);
  __bf16* tiles = reinterpret_cast<__bf16*>(a.partial);
  float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(a.partial) +
                                         round_up((int64_t)gauss_tile_bytes(a), 256));
  if (!a.tiles_ready) {
    gauss_stage_kernel<<<dim3((unsigned)nchunks, (unsigned)ceil_div(cols, kNT)), kStageThreads,
                         0, s>>>(a.N, a.d, static_cast<const float*>(a.X), a.ldx,
                                 static_cast<const float*>(a.Y), nchunks, tiles);
    SLSE_LAUNCH_CHECK();
  }
  // blockIdx.x is the sketch-row block: the blocks that read the same data
  // rows and columns run side by side and share them through the caches
  const int ncb = (int)ceil_div(cols, kNT);
  const int ct = ncb > 1 ? kNT / 64 : (int)ceil_div(cols, 64);
  auto go = [&](auto c, auto r) {
    constexpr int CT = decltype(c)::value, RT = decltype(r)::value;
    dim3 grid((unsigned)ceil_div(a.m, 16 * RT), (unsigned)ncb, (unsigned)a.splits);
    gauss_mfma_kernel<CT, RT><<<grid, kGThreads, 0, s>>>(a.N, a.d, tiles, nchunks, a.seed,
                                                         a.stream_id, a.m, a.splits, part, ldp);
  };
  using std::integral_constant;
  // 128 sketch rows per block halve the copies of [X|Y] per entry of G: taken
  // at 193..320 columns (2^20 x 256: 4.42 ms per pair of 1536 rows against 4.70
  // with 64 rows) where the chip stays full.  Narrower blocks fit a CU twice with
  // 64 rows, which gains more (2^20 x 128: 2.02 against 2.19 ms); wider ones have
  // no registers for 128 rows' accumulators.
  const bool tall = (ct == 4 || ct == 5) && ceil_div(a.m, 128) * a.splits >= 512;
  const integral_constant<int, 4> r4{};
  const integral_constant<int, 8> r8{};
  switch (ct) {
    case 1: go(integral_constant<int, 1>{}, r4); break;
    case 2: go(integral_constant<int, 2>{}, r4); break;
    case 3: go(integral_constant<int, 3>{}, r4); break;
    case 4: tall ? go(integral_constant<int, 4>{}, r8) : go(integral_constant<int, 4>{}, r4); break;
    case 5: tall ? go(integral_constant<int, 5>{}, r8) : go(integral_constant<int, 5>{}, r4); break;
    case 6:
    case 7: go(integral_constant<int, 7>{}, r4); break;
    default: go(integral_constant<int, 9>{}, r4);
  }
  SLSE_LAUNCH_CHECK();
  gauss_reduce_kernel<float, float><<<grid1(a.m * cols), 256, 0, s>>>(
      part, a.splits, a.m, cols, ldp, static_cast<float*>(a.A), a.lda);
  SLSE_LAUNCH_CHECK();
}

// Column tiles of 16 per block of the FP32 / FP64 kernel: every column in one
// block up to 17 tiles in FP32 and 13 in FP64, the widest that are built, else the least
// number of equal blocks; then the next width that is built.  LDS does not set these
// limits (two tiles of the data beside those of G take 104 and 140 KB of 160; 29 and 15
// tiles would fit), and beyond them G is drawn again for every column block: with widths of
// 21, 25 and 29 (FP32) and 15 (FP64) built as well, 4096 rows of 16384 x 400 float32 took
// 1212 us against 1483, 3584 of 65536 x 239 float64 3.89 ms against 4.50.  Products of
// tiles past the columns are wasted, so the widths lie close together.
constexpr int kGaussTiles[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 13, 16, 17};
struct GaussCols {
  int tiles;   // per block
  int blocks;
  bool y_apart;
};
GaussCols gauss_cols(int d, slse_dtype t) {
  auto split = [t](int cols) {
    const int nt = (int)ceil_div(cols, 16);
    const int most = t == SLSE_F64 ? 13 : 17;
    const int want = (int)ceil_div(nt, ceil_div(nt, most));
    GaussCols g{most, 0, false};
    for (int w : kGaussTiles)
      if (w >= want) {
        g.tiles = std::min(w, most);
        break;
      }
    g.blocks = (int)ceil_div(cols, 16 * g.tiles);
    return g;
  };
  const GaussCols with_y = split(d + 1);
  GaussCols g = split(d);
  // Y apart only where that leaves fewer tiles to multiply (elsewhere it costs up to
  // 2.5%: 30000 x 17 FP64 138 and 142 us, 16384 x 512 5990 and 6075)
  g.y_apart = g.blocks * g.tiles < with_y.blocks * with_y.tiles;
  return g.y_apart ? g : with_y;
}
// Sketch rows per block: 128, or 64 where that leaves less of the last block
// empty (few rows: what is drawn past m is skipped, but its waves idle)
int gauss_waves(int64_t m) { return ceil_div(m, 64) % 2 == 1 && m < 512 ? 4 : 8; }

template <typename T, int NT, bool YV>
void gauss_launch(const GaussianArgs& a, const GaussCols& g, T* part, int64_t ldp, hipStream_t s) {
  const int nw = gauss_waves(a.m);
  const int64_t per = ceil_div(a.N, (int64_t)a.splits);
  const int64_t sub_per = round_up(ceil_div(per, (int64_t)a.sub), kGK);
  const dim3 grid((unsigned)ceil_div(a.m, 16 * nw), (unsigned)g.blocks, (unsigned)(a.splits * a.sub));
  const T* X = static_cast<const T*>(a.X);
  const T* Y = static_cast<const T*>(a.Y);
  if (nw == 8)
    gauss_kernel<T, NT, 8, YV><<<grid, 512, 0, s>>>(a.N, a.d, X, a.ldx, Y, a.seed, a.stream_id, a.m,
                                                   a.splits, a.sub, per, sub_per, part, ldp);
  else
    gauss_kernel<T, NT, 4, YV><<<grid, 256, 0, s>>>(a.N, a.d, X, a.ldx, Y, a.seed, a.stream_id, a.m,
                                                   a.splits, a.sub, per, sub_per, part, ldp);
  SLSE_LAUNCH_CHECK();
}

template <typename T, int NT>
void gauss_launch_y(const GaussianArgs& a, const GaussCols& g, T* part, int64_t ldp, hipStream_t s) {
  if (g.y_apart)
    gauss_launch<T, NT, true>(a, g, part, ldp, s);
  else
    gauss_launch<T, NT, false>(a, g, part, ldp, s);
}

template <typename T>
void gaussian_t(const GaussianArgs& a, hipStream_t s) {
  const int cols = a.d + 1;
  const int64_t ldp = round_up(cols, 4);
  T* part = sizeof(T) == 8 ? reinterpret_cast<T*>(a.partial64) : reinterpret_cast<T*>(a.partial);
  const GaussCols g = gauss_cols(a.d, a.t);
  switch (g.tiles) {
#define SLSE_TILES(W) \
  case W: gauss_launch_y<T, W>(a, g, part, ldp, s); break;
    SLSE_TILES(1)
    SLSE_TILES(2)
    SLSE_TILES(3)
    SLSE_TILES(4)
    SLSE_TILES(5)
    SLSE_TILES(6)
    SLSE_TILES(7)
    SLSE_TILES(8)
    SLSE_TILES(9)
    SLSE_TILES(11)
    SLSE_TILES(13)
#undef SLSE_TILES
    default:
      if constexpr (sizeof(T) == 4) {
        if (g.tiles == 16)
          gauss_launch_y<T, 16>(a, g, part, ldp, s);
        else
          gauss_launch_y<T, 17>(a, g, part, ldp, s);
      }
  }
  gauss_reduce_kernel<T, T><<<grid1(a.m * cols), 256, 0, s>>>(part, a.splits * a.sub, a.m, cols, ldp,
                                                               static_cast<T*>(a.A), a.lda);
  SLSE_LAUNCH_CHECK();
}

}  // namespace

size_t countsketch_scratch_bytes(const CountSketchArgs& a) { return cs_scratch(a).bytes; }

void launch_countsketch(const CountSketchArgs& a, hipStream_t s) {
  if (!a.scratch) fail(SLSE_EINVAL, "countsketch: no scratch buffer");
  if (a.t == SLSE_F64)
    countsketch_t<double>(a, s);
  else if (a.t == SLSE_F32)
    countsketch_t<float>(a, s);
  else
    fail(SLSE_EUNSUPPORTED, "countsketch: dtype");
}

void gaussian_plan(GaussianArgs& a) {
  const int64_t tiles = a.bf16 ? ceil_div(a.d + 1, kNT) * ceil_div(a.m, kMT)
                               : ceil_div(a.d + 1, kGT) * ceil_div(a.m, kGT);
  // enough blocks to fill the chip, each split at least a few thousand rows
  int64_t splits = std::max<int64_t>(1, 2048 / std::max<int64_t>(tiles, 1));
  splits = std::min<int64_t>(splits, std::max<int64_t>(1, a.N / 4096));
  a.splits = (int)splits;
  a.sub = 1;
  if (!a.bf16) {
    // the FP32 / FP64 kernel's blocks are large: sub-ranges of a split (at least
    // 256 rows) until there are two per CU
    const int64_t blocks = (int64_t)gauss_cols(a.d, a.t).blocks *
                           ceil_div(a.m, 16 * gauss_waves(a.m)) * splits;
    const int64_t rows = ceil_div(std::max<int64_t>(a.N, 1), splits);
    a.sub = (int)std::max<int64_t>(
        1, std::min<int64_t>(ceil_div(512, std::max<int64_t>(blocks, 1)), rows / 256));
  }
}

size_t gaussian_scratch_bytes(const GaussianArgs& a) {
  const size_t t = gauss_tile_bytes(a);
  return t ? (size_t)round_up((int64_t)t, 256) + gauss_partial_bytes(a) : gauss_partial_bytes(a);
}

void launch_gaussian(const GaussianArgs& a, hipStream_t s) {
  if (a.bf16) {
    if (a.t != SLSE_F32) fail(SLSE_EUNSUPPORTED, "gaussian: BF16 products need F32 data");
    gaussian_mfma(a, s);
    return;
  }
  if (a.t == SLSE_F64)
    gaussian_t<double>(a, s);
  else if (a.t == SLSE_F32)
    gaussian_t<float>(a, s);
  else
    fail(SLSE_EUNSUPPORTED, "gaussian: dtype");
}

void launch_gauss_generate(uint64_t seed, uint64_t stream_id, int64_t m, int64_t N, int blocks,
                           unsigned* sink, hipStream_t s) {
  gauss_generate_kernel<<<blocks, 256, 0, s>>>(seed, stream_id, ceil_div(m, 8), N, sink);
  SLSE_LAUNCH_CHECK();
}

void launch_debug_gaussian(uint64_t seed, uint64_t stream_id, int64_t k0, int64_t nk, int64_t j0,
                           int64_t nj, int form, double* out, hipStream_t s) {
  if (nk * nj <= 0) return;
  debug_gauss_kernel<<<grid1(nk * nj), 256, 0, s>>>(seed, stream_id, k0, nk, j0, nj, form, out);
  SLSE_LAUNCH_CHECK();
}

}  // namespace slse
