// Convergence metrics of Sec. 4.1 on the device: whitening of recorded draws, projections onto the
// fixed directions, merge sorts and the sums of the 1-d Wasserstein distances, and the order
// statistics of the credible limits.  The d x d algebra of the R - 1 statistic runs on the host.
#include <vector>

#include "aux.hpp"

namespace best {
namespace {

constexpr int kMetThreads = 256;

// z[i * zp + it] for draw it = t * N + c of a record [T][d][N]: the draw itself, or with
// mu != nullptr its whitened coordinates, L z = x - mu by forward substitution.  The coordinates
// stay in registers (D: d rounded up to a multiple of 8), so the kernel is bound by its
// 12 d bytes per draw: 27 x 1048576 draws 95 us, against 600 us when earlier coordinates were
// read back from z.
template <int D>
__global__ __launch_bounds__(kMetThreads) void whiten_points_kernel(const float* rec, int64_t T,
                                                                    int d, int64_t N,
                                                                    const double* mu,
                                                                    const double* L, double* z,
                                                                    int64_t zp) {
  const int64_t n = T * N;
  for (int64_t it = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; it < n;
       it += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = it / N, c = it % N;
    double r[D];
#pragma unroll
    for (int i = 0; i < D; ++i) r[i] = (double)rec[(t * d + (i < d ? i : d - 1)) * N + c];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      if (i < d) {
        if (mu) {
          r[i] -= mu[i];
#pragma unroll
          for (int j = 0; j < D; ++j)
            if (j < i) r[i] -= L[i * d + j] * r[j];
          r[i] /= L[i * d + i];
        }
        z[i * zp + it] = r[i];
      }
    }
  }
}

// out[p] = sum over blocks b of part[b * np + p]: 8 interleaved runs of blocks per component,
// combined in order.
__global__ void sum_parts_kernel(const double* part, int nblocks, int np, double* out) {
  __shared__ double sh[8][32];
  const int l = threadIdx.x & 31, q = threadIdx.x >> 5, p = blockIdx.x * 32 + l;
  double s = 0;
  if (p < np) {
#pragma unroll 4
    for (int b = q; b < nblocks; b += 8) s += part[(int64_t)b * np + p];
  }
  sh[q][l] = s;
  __syncthreads();
  if (q == 0 && p < np) {
    s = 0;
    for (int w = 0; w < 8; ++w) s += sh[w][l];
    out[p] = s;
  }
}

// Unit direction k: the d normals of Philox counter (k, 0, stream 6, 0), normalised.
__global__ void directions_kernel(Rng rng, int d, int K, double* w) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  double nrm = 0;
  for (int i = 0; i < d; ++i) {
    const double xi = normal_dim(rng, (uint64_t)k, 0, kStreamProj, 0, i);
    w[k * d + i] = xi;
    nrm += xi * xi;
  }
  nrm = sqrt(nrm);
  for (int i = 0; i < d; ++i) w[k * d + i] /= nrm;
}

// Order-preserving integer image of a double (all NaN above or below every number).
__device__ __forceinline__ uint64_t to_key(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  return (b >> 63) ? ~b : b | 0x8000000000000000ull;
}
__device__ __forceinline__ double from_key(uint64_t k) {
  return __builtin_bit_cast(double, (k >> 63) ? k & 0x7FFFFFFFFFFFFFFFull : ~k);
}

// keys[p * kp + j] = w_p . z_j, kProj directions per thread and point: the point's coordinates
// are read once for them and stay in registers, the directions are zero-padded rows in LDS (as
// scalar loads, each waited for, 128 x 32768 projections in 27 dimensions took 37 us, now 25).
constexpr int kProj = 4;
template <int D>
__global__ __launch_bounds__(kMetThreads) void project_kernel(const double* z, int d, int64_t n,
                                                              int64_t zp, const double* w, int P,
                                                              uint64_t* keys, int64_t kp) {
  __shared__ double ws[kProj][D];
  const int64_t j = blockIdx.x * (int64_t)kMetThreads + threadIdx.x;
  const int p0 = blockIdx.y * kProj;
  for (int e = threadIdx.x; e < kProj * D; e += kMetThreads) {
    const int p = p0 + e / D, i = e % D;
    ws[e / D][i] = p < P && i < d ? w[p * d + i] : 0.0;
  }
  __syncthreads();
  if (j >= n) return;
  double zz[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const double v = z[(int64_t)(i < d ? i : d - 1) * zp + j];
    zz[i] = i < d ? v : 0.0;
  }
#pragma unroll
  for (int p = 0; p < kProj; ++p) {
    double s = 0;
#pragma unroll
    for (int i = 0; i < D; ++i) s += ws[p][i] * zz[i];
    if (p0 + p < P) keys[(p0 + p) * kp + j] = to_key(s);
  }
}

// ---------------------------------------------------------------------------------------
// Merge sort of many independent runs at once.  A tile of kSortTile keys is sorted by one
// workgroup (16 keys per thread in registers, then merges through LDS), and each merge pass
// doubles the sorted length, a workgroup producing kSortTile outputs from the two input ranges that
// a merge-path search finds.  All projections of a batch go through each launch, so a pass is
// bound by its 16 bytes per key instead of by launch latency: 500 projections of 2 x 32768 draws
// take 1.0 ms for everything after the projection; one library sort, scan and sum per
// projection took 47 ms.
// ---------------------------------------------------------------------------------------
constexpr int kSortE = 16;                         // keys per thread
constexpr int kSortTile = kMetThreads * kSortE;    // 4096
constexpr int kSortLds = kSortTile + kSortTile / 16;
// LDS slot of key i: one pad per 16 keeps the blocked accesses of a wave on distinct banks
__device__ __forceinline__ int slot(int i) { return i + (i >> 4); }

// The number of keys that the first k outputs of merging A (na keys) and B (nb) take from A,
// A first on ties; one thread, keys read through `at`.
template <class FA, class FB>
__device__ __forceinline__ int merge_split(int k, int na, int nb, const FA& A, const FB& B) {
  int lo = k > nb ? k - nb : 0, hi = k < na ? k : na;
  while (lo < hi) {
    const int m = (lo + hi) >> 1;
    if (A(m) <= B(k - 1 - m)) lo = m + 1;
    else hi = m;
  }
  return lo;
}

// The same by one wave on arrays in memory: 64 probes per step.
__device__ __forceinline__ int64_t merge_split_wave(int64_t k, const uint64_t* A, int64_t na,
                                                    const uint64_t* B, int64_t nb) {
  const int lane = threadIdx.x & 63;
  int64_t lo = k > nb ? k - nb : 0, hi = k < na ? k : na;
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) / 64, m = lo + (lane + 1) * step - 1;
    const bool in = m < hi;
    const bool less = in && A[in ? m : lo] <= B[k - 1 - (in ? m : lo)];
    const int c = __popcll(__ballot(less)), probes = __popcll(__ballot(in));
    const int64_t l2 = lo + c * step;
    hi = c < probes ? lo + (c + 1) * step - 1 : hi;
    lo = l2;
  }
  return lo;
}

// Sixteen consecutive outputs (from output k) of merging the LDS ranges [a0, a0 + na) and
// [b0, b0 + nb); outputs past the end are not written.
__device__ __forceinline__ void merge_serial(const uint64_t* s, int a0, int na, int b0, int nb,
                                             int k, uint64_t (&o)[kSortE]) {
  int i = merge_split(k, na, nb, [&](int m) { return s[slot(a0 + m)]; },
                      [&](int m) { return s[slot(b0 + m)]; });
  int j = k - i;
  uint64_t x = i < na ? s[slot(a0 + i)] : ~0ull, y = j < nb ? s[slot(b0 + j)] : ~0ull;
#pragma unroll
  for (int u = 0; u < kSortE; ++u) {
    const bool ta = j >= nb || (i < na && x <= y);
    o[u] = ta ? x : y;
    if (ta) {
      ++i;
      x = i < na ? s[slot(a0 + i)] : ~0ull;
    } else {
      ++j;
      y = j < nb ? s[slot(b0 + j)] : ~0ull;
    }
  }
}

// A batch of P projections, each a run of na and a run of nb keys: run r of projection p and its
// tiles, numbered over (p, run, tile).
struct SortBatch {
  int64_t na, nb, pitch;
  int ta, tb;  // tiles of kSortTile keys of the two runs
};
__device__ __forceinline__ void batch_tile(const SortBatch& b, int64_t blk, int64_t& off,
                                           int64_t& len, int& tile) {
  const int per = b.ta + b.tb;
  const int64_t p = blk / per;
  const int t = (int)(blk % per);
  const bool second = t >= b.ta;
  off = p * b.pitch + (second ? b.na : 0);
  len = second ? b.nb : b.na;
  tile = second ? t - b.ta : t;
}

__global__ __launch_bounds__(kMetThreads) void tile_sort_kernel(const uint64_t* in, uint64_t* out,
                                                                SortBatch b) {
  __shared__ uint64_t s[kSortLds];
  int64_t off, len;
  int tile;
  batch_tile(b, blockIdx.x, off, len, tile);
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)tile * kSortTile;
  const int cnt = (int)min((int64_t)kSortTile, len - base);
  const uint64_t* src = in + off + base;
  uint64_t v[kSortE];
#pragma unroll
  for (int u = 0; u < kSortE; ++u) {
    const int i = tid + u * kMetThreads;
    v[u] = i < cnt ? src[i] : ~0ull;  // the padding sorts last
  }
  // Batcher's odd-even merge sort of the thread's 16 keys
#pragma unroll
  for (int p = 1; p < kSortE; p *= 2)
#pragma unroll
    for (int k = p; k >= 1; k /= 2)
#pragma unroll
      for (int j = k % p; j + k < kSortE; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i) {
          if (i + j + k < kSortE && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
            const uint64_t x = v[i + j], y = v[i + j + k];
            const bool sw = y < x;
            v[i + j] = sw ? y : x;
            v[i + j + k] = sw ? x : y;
          }
        }
#pragma unroll
  for (int u = 0; u < kSortE; ++u) s[slot(tid * kSortE + u)] = v[u];
  for (int r = 0; (kSortE << r) < kSortTile; ++r) {
    __syncthreads();
    const int run = kSortE << r, g = tid >> (r + 1), a0 = g * 2 * run;
    merge_serial(s, a0, run, a0 + run, run, (tid & ((2 << r) - 1)) * kSortE, v);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortE; ++u) s[slot(tid * kSortE + u)] = v[u];
  }
  __syncthreads();
  uint64_t* dst = out + off + base;
#pragma unroll
  for (int u = 0; u < kSortE; ++u) {
    const int i = tid + u * kMetThreads;
    if (i < cnt) dst[i] = s[slot(i)];
  }
}

// The input ranges of outputs [k0, k1) of merging A and B, copied to LDS (A's part first): their
// starts and counts.
struct MergeRange {
  int64_t a, b;
  int na, nb;
};
__device__ __forceinline__ MergeRange load_range(const uint64_t* A, int64_t na, const uint64_t* B,
                                                 int64_t nb, int64_t k0, int64_t k1, uint64_t* s,
                                                 int64_t* ends) {
  const int tid = threadIdx.x, wv = tid >> 6;
  if (wv < 2) {
    const int64_t m = merge_split_wave(wv ? k1 : k0, A, na, B, nb);
    if ((tid & 63) == 0) ends[wv] = m;
  }
  __syncthreads();
  MergeRange r;
  r.a = ends[0];
  r.b = k0 - r.a;
  r.na = (int)(ends[1] - r.a);
  r.nb = (int)(k1 - k0) - r.na;
#pragma unroll
  for (int u = 0; u < kSortE; ++u) {
    const int i = tid + u * kMetThreads;
    if (i < r.na) s[slot(i)] = A[r.a + i];
    else if (i < r.na + r.nb) s[slot(i)] = B[r.b + i - r.na];
  }
  __syncthreads();
  return r;
}

// One merge pass: sorted lengths `run` -> 2 run.
__global__ __launch_bounds__(kMetThreads) void merge_pass_kernel(const uint64_t* in, uint64_t* out,
                                                                 SortBatch b, int64_t run) {
  __shared__ uint64_t s[kSortLds];
  __shared__ int64_t ends[2];
  int64_t off, len;
  int tile;
  batch_tile(b, blockIdx.x, off, len, tile);
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)tile * kSortTile, pair = base / (2 * run) * (2 * run);
  const int64_t na = min(run, len - pair), nb = max((int64_t)0, min(run, len - pair - run));
  const int64_t k0 = base - pair, k1 = min(k0 + kSortTile, na + nb);
  const uint64_t* A = in + off + pair;
  const MergeRange r = load_range(A, na, A + run, nb, k0, k1, s, ends);
  uint64_t v[kSortE];
  const int cnt = (int)(k1 - k0);
  if (tid * kSortE < cnt) merge_serial(s, 0, r.na, r.na, r.nb, tid * kSortE, v);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSortE; ++u)
    if (tid * kSortE + u < cnt) s[slot(tid * kSortE + u)] = v[u];
  __syncthreads();
  uint64_t* dst = out + off + base;
#pragma unroll
  for (int u = 0; u < kSortE; ++u) {
    const int i = tid + u * kMetThreads;
    if (i < cnt) dst[i] = s[slot(i)];
  }
}

// Partial sums of |F_a - F_b| (v_{k+1} - v_k) over the merged order of a projection's two sorted
// runs: part[p * nblk + blk] for outputs [blk kSortTile, ..).  After position k, ca values of a and
// cb = k + 1 - ca of b are <= v_k; |ca / na - cb / nb| = |ca nb - cb na| / (na nb), the numerator
// exact in 64-bit integers (both counts below 2^31).
__global__ __launch_bounds__(kMetThreads) void w1_partial_kernel(const uint64_t* keys,
                                                                 SortBatch b, int nblk,
                                                                 double* part) {
  __shared__ uint64_t s[kSortLds];
  __shared__ int64_t ends[2];
  __shared__ double red[kMetThreads];
  const int tid = threadIdx.x, blk = blockIdx.x % nblk;
  const int64_t p = blockIdx.x / nblk, na = b.na, nb = b.nb, n = na + nb;
  const uint64_t* A = keys + p * b.pitch;
  const uint64_t* B = A + na;
  const int64_t k0 = (int64_t)blk * kSortTile, k1 = min(k0 + kSortTile, n);
  const MergeRange r = load_range(A, na, B, nb, k0, k1, s, ends);
  const int k = tid * kSortE, cnt = (int)(k1 - k0);
  const double rn = 1.0 / ((double)na * (double)nb);
  double acc = 0;
  if (k < cnt) {
    int i = merge_split(k, r.na, r.nb, [&](int m) { return s[slot(m)]; },
                        [&](int m) { return s[slot(r.na + m)]; });
    int j = k - i;
    // the heads of both ranges: from LDS, past the block's ranges from memory, ~0 at the end
    auto head_a = [&](int m) {
      return m < r.na ? s[slot(m)] : r.a + m < na ? A[r.a + m] : ~0ull;
    };
    auto head_b = [&](int m) {
      return m < r.nb ? s[slot(r.na + m)] : r.b + m < nb ? B[r.b + m] : ~0ull;
    };
    uint64_t x = head_a(i), y = head_b(j);
    uint64_t cur = 0;
    for (int u = 0; u <= kSortE && k + u <= cnt; ++u) {
      const int64_t ca = r.a + i, cb = r.b + j;
      if (ca + cb >= n) break;  // no next value
      const bool ta = cb >= nb || (ca < na && x <= y);
      const uint64_t next = ta ? x : y;
      if (u > 0)
        acc += (double)llabs(ca * nb - cb * na) * rn * (from_key(next) - from_key(cur));
      cur = next;
      if (ta) x = head_a(++i);
      else y = head_b(++j);
    }
  }
  red[tid] = acc;
  __syncthreads();
  for (int o = kMetThreads / 2; o > 0; o >>= 1) {
    if (tid < o) red[tid] += red[tid + o];
    __syncthreads();
  }
  if (tid == 0) part[p * nblk + blk] = red[0];
}

// out[p] = sum over the projection's nblk partial sums (one workgroup each, fixed order)
__global__ void w1_sum_kernel(const double* part, int nblk, double* out) {
  __shared__ double red[kMetThreads];
  double v = 0;
  for (int i = threadIdx.x; i < nblk; i += kMetThreads) v += part[(int64_t)blockIdx.x * nblk + i];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = kMetThreads / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------------------------------
// Order statistics by radix selection: four ranks (two pairs of neighbours) per parameter, 11 bits
// of the key per pass.  A pass counts the digits of the keys that share a rank's prefix in LDS and
// adds them to the parameter's histograms; the next kernel walks a histogram to the digit that
// holds the rank.  After two passes the keys that share a rank's 22 bits are usually few: they are
// gathered and ranked directly (three reads of the draws in all); where a prefix still holds more
// than kSelCap keys (ties, narrow spreads) the passes go on to the last bit.  Bound by the reads:
// 27 x 1048576 draws 230 us, where sorting every parameter took 5600 us.
// ---------------------------------------------------------------------------------------
constexpr int kSelBits = 11, kSelBins = 1 << kSelBits, kSelPasses = 6, kSelRanks = 4, kSelCap = 2048;
__host__ __device__ constexpr int sel_shift(int pass) {
  return pass + 1 < kSelPasses ? 64 - kSelBits * (pass + 1) : 0;
}
struct SelTarget {
  uint64_t prefix;  // the digits found so far, in place
  int64_t rank;     // the rank among the keys with that prefix
  int64_t count;    // how many keys have it
};

// Calls f(r, key) for every key of the row whose leading bits are those of rank r's prefix, once
// per distinct prefix (psh: shift of the digits found so far).
template <class F>
__device__ __forceinline__ void sel_scan(const double* z, int64_t n, const SelTarget* tg, int psh,
                                         const F& f) {
  uint64_t pre[kSelRanks];
  bool own[kSelRanks];
#pragma unroll
  for (int r = 0; r < kSelRanks; ++r) {
    pre[r] = tg[r].prefix >> psh;
    own[r] = r == 0 || pre[r] != pre[r ? r - 1 : 0];
  }
#pragma unroll 4
  for (int64_t e = blockIdx.x * (int64_t)kMetThreads + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * kMetThreads) {
    const uint64_t k = to_key(z[e]), kp = k >> psh;
#pragma unroll
    for (int r = 0; r < kSelRanks; ++r)
      if (own[r] && kp == pre[r]) f(r, k);
  }
}
// The rank that owns rank r's prefix (the first of a run of equal prefixes).
__device__ __forceinline__ int sel_owner(const SelTarget* tg, int r, int psh) {
  while (r > 0 && tg[r - 1].prefix >> psh == tg[r].prefix >> psh) --r;
  return r;
}

__global__ __launch_bounds__(kMetThreads) void select_count_kernel(const double* z, int64_t n,
                                                                   const SelTarget* tg,
                                                                   unsigned* hist, int pass) {
  __shared__ unsigned h[kSelRanks * kSelBins];
  const int i = blockIdx.y;
  for (int e = threadIdx.x; e < kSelRanks * kSelBins; e += kMetThreads) h[e] = 0;
  __syncthreads();
  const int sh = sel_shift(pass);
  const int width = pass + 1 < kSelPasses ? kSelBits : 64 - kSelBits * (kSelPasses - 1);
  const unsigned mask = (1u << width) - 1;
  if (pass == 0) {
    const double* x = z + (int64_t)i * n;
#pragma unroll 4
    for (int64_t e = blockIdx.x * (int64_t)kMetThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kMetThreads)
      atomicAdd(&h[(unsigned)(to_key(x[e]) >> sh)], 1u);
  } else {
    sel_scan(z + (int64_t)i * n, n, tg + i * kSelRanks, sel_shift(pass - 1), [&](int r, uint64_t k) {
      atomicAdd(&h[r * kSelBins + ((unsigned)(k >> sh) & mask)], 1u);
    });
  }
  __syncthreads();
  unsigned* H = hist + (int64_t)i * kSelRanks * kSelBins;
  for (int e = threadIdx.x; e < kSelRanks * kSelBins; e += kMetThreads)
    if (h[e]) atomicAdd(&H[e], h[e]);
}

// One workgroup per parameter: the digit of every rank; clears the histograms for the next pass.
__global__ __launch_bounds__(kMetThreads) void select_digit_kernel(unsigned* hist, SelTarget* tg_all,
                                                                   int pass) {
  __shared__ int64_t run[kMetThreads];
  __shared__ SelTarget next[kSelRanks];
  const int tid = threadIdx.x;
  constexpr int per = kSelBins / kMetThreads;
  unsigned* H = hist + (int64_t)blockIdx.x * kSelRanks * kSelBins;
  SelTarget* tg = tg_all + blockIdx.x * kSelRanks;
  for (int r = 0; r < kSelRanks; ++r) {
    const int own = pass ? sel_owner(tg, r, sel_shift(pass - 1)) : 0;
    unsigned c[per];
    int64_t s = 0;
#pragma unroll
    for (int u = 0; u < per; ++u) {
      c[u] = H[own * kSelBins + tid * per + u];
      s += c[u];
    }
    run[tid] = s;
    __syncthreads();
    for (int o = 1; o < kMetThreads; o <<= 1) {
      const int64_t v = tid >= o ? run[tid - o] : 0;
      __syncthreads();
      run[tid] += v;
      __syncthreads();
    }
    int64_t before = run[tid] - s;
    const int64_t rank = tg[r].rank;
    if (rank >= before && rank < before + s) {
      int digit = 0;
      unsigned cnt = c[0];
#pragma unroll
      for (int u = 0; u + 1 < per; ++u) {
        if (digit == u && rank >= before + c[u]) {
          before += c[u];
          digit = u + 1;
          cnt = c[u + 1];
        }
      }
      next[r] = SelTarget{tg[r].prefix | (uint64_t)(tid * per + digit) << sel_shift(pass),
                          rank - before, cnt};
    }
    __syncthreads();
  }
  if (tid < kSelRanks) tg[tid] = next[tid];
  for (int e = tid; e < kSelRanks * kSelBins; e += kMetThreads) H[e] = 0;
}

// The keys with a rank's 22-bit prefix, in any order; len[rank] their number.
__global__ __launch_bounds__(kMetThreads) void select_gather_kernel(const double* z, int64_t n,
                                                                    const SelTarget* tg,
                                                                    uint64_t* list, unsigned* len) {
  const int i = blockIdx.y;
  sel_scan(z + (int64_t)i * n, n, tg + i * kSelRanks, sel_shift(1), [&](int r, uint64_t k) {
    const unsigned at = atomicAdd(&len[i * kSelRanks + r], 1u);
    if (at < kSelCap) list[(int64_t)(i * kSelRanks + r) * kSelCap + at] = k;
  });
}

// One workgroup per (parameter, rank): the gathered key of that rank (or, with list = nullptr, the
// finished prefix) as a value.
__global__ __launch_bounds__(kMetThreads) void select_value_kernel(const SelTarget* tg,
                                                                   const uint64_t* list,
                                                                   double* out) {
  __shared__ uint64_t s[kSelCap];
  const int b = blockIdx.x, i = b / kSelRanks;
  if (!list) {
    if (threadIdx.x == 0) out[b] = from_key(tg[b].prefix);
    return;
  }
  const int own = i * kSelRanks + sel_owner(tg + i * kSelRanks, b % kSelRanks, sel_shift(1));
  const int m = (int)tg[b].count;
  for (int e = threadIdx.x; e < m; e += kMetThreads) s[e] = list[(int64_t)own * kSelCap + e];
  __syncthreads();
  for (int e = threadIdx.x; e < m; e += kMetThreads) {
    const uint64_t k = s[e];
    int64_t below = 0;
    for (int q = 0; q < m; ++q) below += s[q] < k || (s[q] == k && q < e);
    if (below == tg[b].rank) out[b] = from_key(k);
  }
}

__global__ void sel_clear_kernel(unsigned* hist, int64_t n) {
  for (int64_t e = blockIdx.x * (int64_t)kMetThreads + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * kMetThreads)
    hist[e] = 0;
}

int blocks_for(int64_t n) {
  int64_t g = (n + kMetThreads - 1) / kMetThreads;
  if (g < 1) g = 1;
  if (g > 4096) g = 4096;
  return (int)g;
}

}  // namespace

hipError_t launch_whiten_points(const float* rec, int64_t T, int d, int64_t N, const double* mu,
                                const double* L, double* z, int64_t zpitch, hipStream_t s) {
  const dim3 g(blocks_for(T * N)), b(kMetThreads);
  if (d <= 8) hipLaunchKernelGGL((whiten_points_kernel<8>), g, b, 0, s, rec, T, d, N, mu, L, z, zpitch);
  else if (d <= 16) hipLaunchKernelGGL((whiten_points_kernel<16>), g, b, 0, s, rec, T, d, N, mu, L, z, zpitch);
  else hipLaunchKernelGGL((whiten_points_kernel<kMaxD>), g, b, 0, s, rec, T, d, N, mu, L, z, zpitch);
  return hipGetLastError();
}

hipError_t launch_sum_parts(const double* part, int nblocks, int np, double* out, hipStream_t s) {
  hipLaunchKernelGGL(sum_parts_kernel, dim3((np + 31) / 32), dim3(256), 0, s, part, nblocks, np, out);
  return hipGetLastError();
}

hipError_t launch_directions(const Rng& rng, int d, int K, double* w, hipStream_t s) {
  hipLaunchKernelGGL(directions_kernel, dim3((K + kMetThreads - 1) / kMetThreads),
                     dim3(kMetThreads), 0, s, rng, d, K, w);
  return hipGetLastError();
}

static hipError_t launch_project(const double* z, int d, int64_t n, const double* w, int P,
                                 uint64_t* keys, int64_t kpitch, hipStream_t s) {
  const dim3 g((unsigned)((n + kMetThreads - 1) / kMetThreads), (unsigned)((P + kProj - 1) / kProj)),
      b(kMetThreads);
  if (d <= 8) hipLaunchKernelGGL((project_kernel<8>), g, b, 0, s, z, d, n, n, w, P, keys, kpitch);
  else if (d <= 16) hipLaunchKernelGGL((project_kernel<16>), g, b, 0, s, z, d, n, n, w, P, keys, kpitch);
  else hipLaunchKernelGGL((project_kernel<kMaxD>), g, b, 0, s, z, d, n, n, w, P, keys, kpitch);
  return hipGetLastError();
}

int64_t sliced_w1_parts(int64_t n) { return (n + kSortTile - 1) / kSortTile; }

hipError_t launch_sliced_w1(const double* za, int64_t na, const double* zb, int64_t nb, int d,
                            const double* w, int P, uint64_t* keys, uint64_t* tmp, double* part,
                            double* out, hipStream_t s) {
  const int64_t n = na + nb;
  hipError_t e = launch_project(za, d, na, w, P, keys, n, s);
  if (e == hipSuccess) e = launch_project(zb, d, nb, w, P, keys + na, n, s);
  if (e != hipSuccess) return e;
  const SortBatch b{na, nb, n, (int)((na + kSortTile - 1) / kSortTile),
                    (int)((nb + kSortTile - 1) / kSortTile)};
  const dim3 grid((unsigned)((int64_t)P * (b.ta + b.tb)));
  hipLaunchKernelGGL(tile_sort_kernel, grid, dim3(kMetThreads), 0, s, keys, tmp, b);
  uint64_t *src = tmp, *dst = keys;
  for (int64_t run = kSortTile; run < (na > nb ? na : nb); run *= 2) {
    hipLaunchKernelGGL(merge_pass_kernel, grid, dim3(kMetThreads), 0, s, src, dst, b, run);
    uint64_t* t = src;
    src = dst;
    dst = t;
  }
  const int nblk = (int)sliced_w1_parts(n);
  hipLaunchKernelGGL(w1_partial_kernel, dim3((unsigned)((int64_t)P * nblk)), dim3(kMetThreads), 0, s,
                     src, b, nblk, part);
  hipLaunchKernelGGL(w1_sum_kernel, dim3((unsigned)P), dim3(kMetThreads), 0, s, part, nblk, out);
  return hipGetLastError();
}

size_t select_scratch_bytes(int d) {
  return (size_t)d * kSelRanks * (kSelBins * sizeof(unsigned) + kSelCap * sizeof(uint64_t) +
                                  sizeof(SelTarget) + sizeof(double) + sizeof(unsigned));
}

// The values of ranks[4] (host, ascending) in each of the d rows of z ([d][n]): out (host) [d][4].
hipError_t select_ranks(const double* z, int d, int64_t n, const int64_t* ranks, void* scratch,
                        double* out, hipStream_t s) {
  const int nt = d * kSelRanks;
  uint64_t* list = (uint64_t*)scratch;
  SelTarget* tg = (SelTarget*)(list + (size_t)nt * kSelCap);
  double* val = (double*)(tg + nt);
  unsigned* hist = (unsigned*)(val + nt);
  unsigned* len = hist + (size_t)nt * kSelBins;
  std::vector<SelTarget> host(nt);
  for (int i = 0; i < nt; ++i) host[i] = SelTarget{0, ranks[i % kSelRanks], n};
  const size_t tb = nt * sizeof(SelTarget);
  hipError_t e = hipMemcpyAsync(tg, host.data(), tb, hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sel_clear_kernel, dim3(256), dim3(kMetThreads), 0, s, hist,
                     (int64_t)nt * (kSelBins + 1));
  // blocks of at least 4096 draws: each adds a histogram to memory
  int64_t g = (n + 4095) / 4096;
  const int64_t cap = (2048 + d - 1) / d;
  if (g > cap) g = cap;
  const dim3 grid((unsigned)g, (unsigned)d), thr(kMetThreads);
  bool gather = false;
  for (int p = 0; p < kSelPasses && !gather; ++p) {
    hipLaunchKernelGGL(select_count_kernel, grid, thr, 0, s, z, n, tg, hist, p);
    hipLaunchKernelGGL(select_digit_kernel, dim3((unsigned)d), thr, 0, s, hist, tg, p);
    if (p == 1) {
      if ((e = hipMemcpyAsync(host.data(), tg, tb, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
      if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
      gather = true;
      for (const SelTarget& t : host) gather = gather && t.count <= kSelCap;
    }
  }
  if (gather) hipLaunchKernelGGL(select_gather_kernel, grid, thr, 0, s, z, n, tg, list, len);
  hipLaunchKernelGGL(select_value_kernel, dim3((unsigned)nt), thr, 0, s, tg,
                     gather ? list : (const uint64_t*)nullptr, val);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(out, val, nt * sizeof(double), hipMemcpyDeviceToHost, s)) != hipSuccess)
    return e;
  return hipStreamSynchronize(s);
}

}  // namespace best
