// Non-templated kernels: walker initialisation, re-whitening, dual averaging, statistics,
// ensemble moments + jittered Cholesky (Sec. 3.2), multi-chain autocovariances for ESS, the plain
// model's values, and the training weight-gradient GEMMs.
#include <mutex>
#include <type_traits>

#include "aux.hpp"

namespace best {

// ---- walker initialisation (Sec. 3.2: uniform / replicated / Gaussian / hypersphere) ---
__global__ void init_positions_kernel(Target tg, State S, Rng rng, int mode, const double* pt,
                                      double scale, const double* L0, uint64_t step) {
  const int d = tg.d;
  const int64_t n = (int64_t)d * S.N;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / S.N);
    const int64_t c = e % S.N;
    double v;
    if (mode == 0) {
      const U4 b = rng.block(c, step, kStreamInit, 0, (uint32_t)(i >> 1));
      const double u = (i & 1) ? u52(b.z, b.w) : u52(b.x, b.y);
      v = tg.lower[i] + (tg.upper[i] - tg.lower[i]) * u;
    } else if (mode == 1) {
      v = pt[i];
    } else if (mode == 2) {
      double s = 0;
      for (int j = 0; j <= i; ++j) s += L0[i * d + j] * normal_dim(rng, c, step, kStreamInit, 1, j);
      v = pt[i] + scale * s;
    } else {
      // uniform in the unit ball: direction xi / |xi| from d normals (sub 2), radius U^(1/d)
      // from the first uniform of block 0 of sub 3; then mapped through L0 and scaled
      double nn = 0, s = 0;
      for (int j = 0; j < d; ++j) {
        const double xj = normal_dim(rng, c, step, kStreamInit, 2, j);
        nn += xj * xj;
        if (j <= i) s += L0[i * d + j] * xj;
      }
      const U4 b = rng.block(c, step, kStreamInit, 3, 0);
      const double r = pow(u52(b.x, b.y), 1.0 / (double)d);
      v = pt[i] + scale * r * s / sqrt(nn);
    }
    S.x[i * S.Np + c] = v;
  }
}

// z = L^{-1} (x - mu) by forward substitution, one thread per chain.
__global__ void rewhiten_kernel(State S, Whiten W, int d) {
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < S.N;
       c += (int64_t)gridDim.x * blockDim.x) {
    double zz[kMaxD];
    for (int i = 0; i < d; ++i) {
      double r = S.x[i * S.Np + c] - W.mu[i];
      for (int j = 0; j < i; ++j) r -= W.L[i * d + j] * zz[j];
      zz[i] = r / W.L[i * d + i];
      S.z[i * S.Np + c] = zz[i];
    }
  }
}

// Fixed-order block reduction of a double per thread (256 threads).
__device__ double block_sum(double v, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int s = kAuxThreads / 2; s > 0; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// ---- dual averaging (Hoffman & Gelman 2014) on the chain-mean acceptance -------------
// da = [mu, h_bar, log_eps_bar, m, eps, delta, gamma, t0, kappa]
__global__ void da_update_kernel(const double* step_prob, int64_t N, double* da) {
  __shared__ double sh[kAuxThreads];
  double v = 0;
  for (int64_t c = threadIdx.x; c < N; c += kAuxThreads) v += step_prob[c];
  const double mean = block_sum(v, sh) / (double)N;
  if (threadIdx.x == 0) {
    const double m = da[3] + 1.0;
    const double w = 1.0 / (m + da[7]);
    const double hb = (1.0 - w) * da[1] + w * (da[5] - mean);
    const double log_eps = da[0] - sqrt(m) / da[6] * hb;
    const double eta = pow(m, -da[8]);
    da[1] = hb;
    da[2] = eta * log_eps + (1.0 - eta) * da[2];
    da[3] = m;
    da[4] = exp(log_eps);
  }
}

// ---- per-call statistics: [accepted, nonfinite, oob] int64 + [sum_prob] -----------------
__global__ void stats_kernel(State S, int64_t* out_i, double* out_d) {
  __shared__ double sh[kAuxThreads];
  double a = 0, nf = 0, oob = 0, ne = 0, sp = 0;
  for (int64_t c = threadIdx.x; c < S.N; c += kAuxThreads) {
    a += S.n_acc[c];
    nf += S.n_nonfinite[c];
    oob += S.n_oob[c];
    ne += S.n_evals[c];
    sp += S.sum_prob[c];
  }
  a = block_sum(a, sh);
  nf = block_sum(nf, sh);
  oob = block_sum(oob, sh);
  ne = block_sum(ne, sh);
  sp = block_sum(sp, sh);
  if (threadIdx.x == 0) {
    out_i[0] = (int64_t)a;
    out_i[1] = (int64_t)nf;
    out_i[2] = (int64_t)oob;
    out_i[3] = (int64_t)ne;
    out_d[0] = sp;
  }
}

__global__ void aies_record_kernel(State S, int d, float* rec, int64_t slot, int64_t pitch) {
  const int64_t n = (int64_t)d * S.N;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / S.N);
    const int64_t c = e % S.N;
    rec[(slot * d + i) * pitch + c] = (float)S.x[i * S.Np + c];
  }
}

// ---- ensemble moments, pass 1: per-block shifted sums over items ----------------------
// Items come from a float record [T][d][N] (item = t*N + c) or an FP64 array [d][pitch].
// The shift is one vector s_i (spitch 0) or one per chain, s_i(c) = shift[i*spitch + c].
// Slot p < d holds sum (v_i - s_i); slot d + pair(i, j), j <= i, holds sum of products.
//
// For the covariance adaptation: a thread per slot over blocks of 128 items in LDS.  This order of
// the sums is part of the adapted whitening's bits, hence of every later accept decision, so it
// stays as it is (22 us for 6 x 81920 items, once per window).
__global__ void adapt_moments_kernel(const float* rec, const double* xs, int64_t T, int64_t N,
                                     int64_t pitch, int d, const double* shift, double* part) {
  constexpr int kChunk = 128;
  __shared__ double v[kChunk][kMaxD + 1];
  const int np = d + d * (d + 1) / 2;
  const int64_t items = T * N;
  const int64_t per = (items + gridDim.x - 1) / gridDim.x;
  const int64_t b0 = blockIdx.x * per, b1 = min(items, b0 + per);
  double accs[4] = {0, 0, 0, 0};  // np <= d + d(d+1)/2 = 560 <= 4 * 256
  for (int64_t base = b0; base < b1; base += kChunk) {
    const int64_t it = base + threadIdx.x;
    if (threadIdx.x < kChunk && it < b1) {
      const int64_t t = it / N, c = it % N;
      for (int i = 0; i < d; ++i) {
        const double x = rec ? (double)rec[(t * d + i) * pitch + c] : xs[i * pitch + c];
        v[threadIdx.x][i] = x - shift[i];
      }
    }
    __syncthreads();
    const int cnt = (int)min((int64_t)kChunk, b1 - base);
    for (int k = 0; k < 4; ++k) {
      const int p = threadIdx.x + k * kAuxThreads;
      if (p >= np) break;
      int i, j;
      if (p < d) {
        i = p;
        j = -1;
      } else {
        int q = p - d;
        i = 0;
        while (q > i) {
          q -= i + 1;
          ++i;
        }
        j = q;
      }
      double s = 0;
      if (j < 0) {
        for (int r = 0; r < cnt; ++r) s += v[r][i];
      } else {
        for (int r = 0; r < cnt; ++r) s += v[r][i] * v[r][j];
      }
      accs[k] += s;
    }
    __syncthreads();
  }
  for (int k = 0; k < 4; ++k) {
    const int p = threadIdx.x + k * kAuxThreads;
    if (p < np) part[(int64_t)blockIdx.x * np + p] = accs[k];
  }
}

// For the convergence metrics: the products are V^T V on FP64 MFMA (K = items): a wave takes 16
// chains of one step at a time, a lane four consecutive chains of one parameter, which are its
// operand of four MFMAs as A and as B alike.  D16 is the number of 16-parameter blocks (one product
// tile, or three); VEC: N is a multiple of 4, so a lane's chains are one load.  Bound by the matrix
// rate, 3 x 64 cycles per 4 items at d > 16, and the record's bytes: 27 x 1048576 items 59 us,
// against 670 us with two LDS reads per product.
constexpr int kMomWaves = 16;
template <int D16, bool REC, bool VEC>
__global__ __launch_bounds__(64 * kMomWaves) void moments_partial_kernel(
    const float* rec, const double* xs, int64_t T, int64_t N, int64_t pitch, int d,
    const double* shift, int64_t spitch, double* part) {
  constexpr int NT = D16 * (D16 + 1) / 2;  // product tiles (a, b), b <= a
  __shared__ double sh[NT * 256 + D16 * 16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, cl = lane & 15;
  const int64_t per_t = (N + 15) / 16, chunks = T * per_t;
  f64x4 acc[NT] = {};
  double sum[D16] = {};
  for (int64_t q = blockIdx.x * (int64_t)kMomWaves + wv; q < chunks;
       q += (int64_t)gridDim.x * kMomWaves) {
    const int64_t t = q / per_t, c = (q % per_t) * 16 + 4 * g;
    double v[D16][4];
#pragma unroll
    for (int b = 0; b < D16; ++b) {
      const int i = b * 16 + cl, ii = i < d ? i : d - 1;
      if constexpr (VEC && REC) {
        const bool in = i < d && c < N;
        const int64_t cc = c < N ? c : N - 4;
        float x[4];
        double s[4];
        __builtin_memcpy(x, rec + (t * d + ii) * pitch + cc, 16);
        if (spitch) __builtin_memcpy(s, shift + ii * spitch + cc, 32);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[b][r] = in ? (double)x[r] - (spitch ? s[r] : shift[ii]) : 0.0;
        continue;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t cc = c + r < N ? c + r : N - 1;
        const double x = REC ? (double)rec[(t * d + ii) * pitch + cc] : xs[ii * pitch + cc];
        const double s = spitch ? shift[ii * spitch + cc] : shift[ii];
        v[b][r] = i < d && c + r < N ? x - s : 0.0;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int k = 0;
#pragma unroll
      for (int a = 0; a < D16; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b, ++k)
          acc[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[a][r], v[b][r], acc[k], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < D16; ++b) sum[b] += v[b][r];
    }
  }
#pragma unroll
  for (int b = 0; b < D16; ++b) sum[b] = sum_lane_groups(sum[b]);
  // the waves add their tiles in order; D slot r of a lane is (row g + 4 r, column cl)
  for (int w = 0; w < kMomWaves; ++w) {
    if (wv == w) {
#pragma unroll
      for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double* o = sh + k * 256 + (g + 4 * r) * 16 + cl;
          *o = w ? *o + acc[k][r] : acc[k][r];
        }
      if (g == 0) {
#pragma unroll
        for (int b = 0; b < D16; ++b) {
          double* o = sh + NT * 256 + b * 16 + cl;
          *o = w ? *o + sum[b] : sum[b];
        }
      }
    }
    __syncthreads();
  }
  const int np = d + d * (d + 1) / 2;
  for (int p = tid; p < np; p += 64 * kMomWaves) {
    double v;
    if (p < d) {
      v = sh[NT * 256 + p];
    } else {
      int q = p - d, i = 0;
      while (q > i) {
        q -= i + 1;
        ++i;
      }
      const int a = i >> 4, b = q >> 4;
      v = sh[(a * (a + 1) / 2 + b) * 256 + (i & 15) * 16 + (q & 15)];
    }
    part[(int64_t)blockIdx.x * np + p] = v;
  }
}

// Cholesky factor of a (d x d, row-major, LDS) into L by columns, one thread per row (every thread
// of the workgroup calls; the sums run over k in order); false if a pivot is not finite and above
// `floor` (numerical positive definiteness).
__device__ bool chol(const double* a, double* L, int d, double floor, int* bad) {
  const int i = threadIdx.x;
  for (int e = i; e < d * d; e += kAuxThreads) L[e] = 0;
  if (i == 0) *bad = 0;
  __syncthreads();
  for (int j = 0; j < d; ++j) {
    double s = 0;
    if (i >= j && i < d) {
      s = a[i * d + j];
      for (int k = 0; k < j; ++k) s -= L[i * d + k] * L[j * d + k];
      if (i == j) {
        if (!(s > floor) || !isfinite(s)) *bad = 1;
        L[j * d + j] = sqrt(s);
      }
    }
    __syncthreads();
    if (*bad) break;
    if (i > j && i < d) L[i * d + j] = s / L[j * d + j];
    __syncthreads();
  }
  const bool ok = *bad == 0;
  __syncthreads();
  return ok;
}

// Pass 2 (one block): mean, covariance, symmetrise, jittered Cholesky; on success writes
// the new whitening.  info = [status (0 ok / 1 not PD), jitter, logdet].
// The partial sums are added in block order, sixteen loads ahead.
__global__ __launch_bounds__(kAuxThreads) void moments_final_kernel(
    const double* part, int nblocks, int64_t count, int d, const double* shift, int update_mean,
    double* mu, double* Lout, double* info) {
  constexpr int kMaxP = kMaxD + kMaxD * (kMaxD + 1) / 2;
  __shared__ double S[kMaxD * kMaxD];
  __shared__ double Lt[kMaxD * kMaxD];
  __shared__ double sum[kMaxP];
  __shared__ double diag[kMaxD];
  __shared__ int bad;
  const int tid = threadIdx.x, np = d + d * (d + 1) / 2;
  for (int p = tid; p < np; p += kAuxThreads) {
    double s = 0;
    for (int b0 = 0; b0 < nblocks; b0 += 16) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = part[(int64_t)(b0 + u < nblocks ? b0 + u : b0) * np + p];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (b0 + u < nblocks) s += v[u];
    }
    sum[p] = s;
  }
  __syncthreads();
  const double n = (double)count;
  for (int e = tid; e < d * d; e += kAuxThreads) {
    const int i = e / d > e % d ? e / d : e % d, j = e / d > e % d ? e % d : e / d;
    const double c = (sum[d + i * (i + 1) / 2 + j] - sum[i] * sum[j] / n) / (n - 1.0);
    S[e] = c;
    if (i == j) diag[i] = c;
  }
  __syncthreads();
  double jit = 0, scale = 0;
  for (int i = 0; i < d; ++i) scale += diag[i];
  scale /= d;
  const double floor = isfinite(scale) ? 1e-12 * scale : 0.0;  // pivot floor
  bool ok = chol(S, Lt, d, floor, &bad);
  for (double lam = 1e-10; lam <= 1e-2 * (1 + 1e-12) && !ok; lam *= 10.0) {
    jit = lam * scale;
    if (tid < d) S[tid * d + tid] = diag[tid] + jit;
    __syncthreads();
    ok = chol(S, Lt, d, floor, &bad);
  }
  if (!ok) {
    if (tid == 0) {
      info[0] = 1;
      info[1] = jit;
    }
    return;
  }
  for (int e = tid; e < d * d; e += kAuxThreads) Lout[e] = Lt[e];
  if (update_mean && tid < d) mu[tid] = shift[tid] + sum[tid] / n;
  if (tid == 0) {
    double ld = 0;
    for (int i = 0; i < d; ++i) ld += log(Lt[i * d + i]);
    info[0] = 0;
    info[1] = jit;
    info[2] = ld;
  }
}

// ---- ESS ----------------------------------------------------------------------------------
// Per-chain mean and sum of squared deviations: a workgroup holds 64 chains of one parameter, its
// 16 waves every 16th step each, so a record of few chains still fills the chip.  One pass over the
// record: a wave sums eight values at a time about the first of them (their squares are at most nine
// times the block's deviations), the squares of its blocks are combined by the pairwise formula (Chan,
// Golub & LeVeque 1979),
//   ssq += ssq_b + (mean_b - mean)^2 n n_b / (n + n_b),
// and those of the waves by their distances from the common mean, so that the error is that of two
// passes wherever the chain starts.  (As S2 - S1^2 / T about the chain's first value it grows T times for
// a chain that starts far from its mean.)  Means are taken relative to that first value, from which
// neighbouring floats differ exactly.  Bound by the record's bytes: 4000 x 6 x 4096 (393 MB) 93 us; a
// thread per chain with two passes took 3190 us.  A record of few chains has few workgroups and is bound by
// their FP64 instructions: so the mask stands in the last block alone, the reciprocals of 64 blocks
// are taken by the 64 lanes at once, and two workgroups share a CU (at most 64 VGPRs).  The ESS of 42 x 6
// chains x 3820 steps takes 127 us (142 with a mask and a division in every block), of 900 x 20 x 300 72 us (79).
constexpr int kStatWaves = 16, kStatBlock = 8;
struct StatSteps {  // the first n_split waves have d_hi steps each, the others d_lo, one less
  int n_split;
  double d_hi, d_lo, r_T, r_hi, r_lo, tail_hi, tail_lo;  // r: reciprocals (0 of 0), tail: of the last block's steps
};
__global__ __launch_bounds__(64 * kStatWaves, 8) void ess_chain_stats_kernel(const float* rec,
                                                                          int64_t T, int d,
                                                                          int64_t N, StatSteps n,
                                                                          double* mean,
                                                                          double* ssq) {
  __shared__ double sh[2][kStatWaves][64];
  const int lane = threadIdx.x & 63, i = blockIdx.y;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t st = (int64_t)d * N;
  const int64_t n_w = (T - wv + kStatWaves - 1) / kStatWaves;  // steps of this wave, wv, wv + 16, ..
  for (int64_t cb = blockIdx.x; cb * 64 < N; cb += gridDim.x) {
    const int64_t c = cb * 64 + lane;
    const unsigned cl = (unsigned)(c < N ? lane : N - 1 - cb * 64);
    const float* __restrict__ x = rec + (int64_t)i * N + cb * 64;  // scalar; lane offset cl
    const double x0 = x[cl];
    double s1 = 0, q = 0, rk = 0;  // over the wave's first k values: sum, squares about their mean, 1 / k
    const float* p = x + wv * st;
    double rtab = 0;  // lane l: one over the values up to block l of 64
    int64_t k = 0;
    double kd = 0;  // k
    for (; k + kStatBlock <= n_w; k += kStatBlock) {
      const int kb = (int)(k / kStatBlock) & 63;
      if (kb == 0) rtab = 1.0 / (double)(k + (lane + 1) * kStatBlock);
      float v[kStatBlock];
#pragma unroll
      for (int u = 0; u < kStatBlock; ++u) {
        v[u] = p[cl];
        p += kStatWaves * st;
      }
      const double c0 = v[0];
      double sb = 0, qb = 0;
#pragma unroll
      for (int u = 1; u < kStatBlock; ++u) {
        const double y = (double)v[u] - c0;
        sb += y;
        qb += y * y;
      }
      const double off = c0 - x0, dm = (off + sb * (1.0 / kStatBlock)) - s1 * rk;
      rk = lane_value(rtab, kb);
      q += (qb - sb * (sb * (1.0 / kStatBlock))) + dm * dm * (kd * (double)kStatBlock * rk);
      kd += (double)kStatBlock;
      s1 += off * (double)kStatBlock + sb;
    }
    if (k < n_w) {
      const int nb = (int)(n_w - k);
      float v[kStatBlock];  // the last value again past the end
#pragma unroll
      for (int u = 0; u < kStatBlock; ++u) {
        v[u] = p[cl];
        if (k + u + 1 < n_w) p += kStatWaves * st;
      }
      const double c0 = v[0];
      double sb = 0, qb = 0;
#pragma unroll
      for (int u = 1; u < kStatBlock; ++u) {
        if (u >= nb) break;  // the same in every lane
        const double y = (double)v[u] - c0;
        sb += y;
        qb += y * y;
      }
      const double rb = wv < n.n_split ? n.tail_hi : n.tail_lo, off = c0 - x0;
      const double dm = (off + sb * rb) - s1 * rk;
      q += (qb - sb * (sb * rb)) + dm * dm * (kd * (double)nb * (wv < n.n_split ? n.r_hi : n.r_lo));
      s1 += off * (double)nb + sb;
    }
    sh[0][wv][lane] = s1;
    sh[1][wv][lane] = q;
    __syncthreads();
    if (wv == 0 && c < N) {
      s1 = q = 0;
#pragma unroll 8
      for (int w = 0; w < kStatWaves; ++w) s1 += sh[0][w][lane];  // zero for a wave without steps
      const double m = s1 * n.r_T;
#pragma unroll 8
      for (int w = 0; w < kStatWaves; ++w) {
        const double dm = sh[0][w][lane] * (w < n.n_split ? n.r_hi : n.r_lo) - m;
        q += sh[1][w][lane] + (w < n.n_split ? n.d_hi : n.d_lo) * (dm * dm);
      }
      mean[i * N + c] = x0 + m;
      ssq[i * N + c] = q;
    }
    __syncthreads();
  }
}

// Over the chains of one parameter: out = [sum ssq, mean of the means, sum (mean - that)^2,
// max |mean|] (one workgroup per parameter, fixed order).
__global__ void ess_param_stats_kernel(const double* mean, const double* ssq, int64_t N,
                                       double* out) {
  __shared__ double sh[kAuxThreads];
  const double* m = mean + (int64_t)blockIdx.x * N;
  const double* q = ssq + (int64_t)blockIdx.x * N;
  double w = 0, s = 0, mx = 0;
#pragma unroll 4
  for (int64_t c = threadIdx.x; c < N; c += kAuxThreads) {
    w += q[c];
    s += m[c];
    mx = fmax(mx, fabs(m[c]));
  }
  w = block_sum(w, sh);
  const double mm = block_sum(s, sh) / (double)N;
  double b = 0;
#pragma unroll 4
  for (int64_t c = threadIdx.x; c < N; c += kAuxThreads) {
    const double dm = m[c] - mm;
    b += dm * dm;
  }
  b = block_sum(b, sh);
  sh[threadIdx.x] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int t = 1; t < kAuxThreads; ++t) mx = fmax(mx, sh[t]);
    double* o = out + 4 * blockIdx.x;
    o[0] = w;
    o[1] = mm;
    o[2] = b;
    o[3] = mx;
  }
}

// Sums over chains and steps of y_s y_{s - lag} (y = x - chain mean, zero outside the record) for
// windows of kEssLB lags (LAG0: the window of lags 0 ..).  One wave holds 64 chains of one parameter over one of S time segments:
// a lane keeps its chain's last kEssLB (delayed) values and the kEssLB sums in registers, so a step
// is one load and kEssLB FP64 FMAs without LDS.  Bound by the FP64 rate (and by the record's bytes
// for the first window): 4000 x 6 x 4096, 32 lags 150 us, of which 86 us are the FMAs.  The
// time segments give small ensembles enough waves; with the windows staged through LDS (an LDS
// read per FMA, 128 lags) the first pass took 9100 us.
constexpr int kEssChunk = 16;  // steps loaded together (kEssLB a multiple)
template <bool LAG0>
__global__ __launch_bounds__(64, LAG0 ? 3 : 2) void ess_autocov_kernel(const float* rec, const double* mean,
                                                            int64_t T, int d, int64_t N,
                                                            int64_t lag0, int n_win, int64_t seg,
                                                            double* part) {
  const int lane = threadIdx.x, i = blockIdx.y, win = blockIdx.z % n_win, sg = blockIdx.z / n_win;
  const int n_seg = gridDim.z / n_win;
  const int64_t cb = blockIdx.x, st = (int64_t)d * N;
  const bool valid = cb * 64 + lane < N;
  const unsigned cl = (unsigned)(valid ? lane : N - 1 - cb * 64);  // idle lanes repeat a chain
  const int64_t lag = LAG0 ? 0 : lag0 + (int64_t)win * kEssLB;
  const float* __restrict__ x = rec + (int64_t)i * N + cb * 64;
  const double mc = mean[(int64_t)i * N + cb * 64 + cl];
  const int64_t s0 = sg * seg, s1 = min(T, s0 + seg);
  double acc[kEssLB], w[kEssLB];
#pragma unroll
  for (int k = 0; k < kEssLB; ++k) acc[k] = 0;
  // steps [s, s + kEssChunk), window slots J ..; zeros for the steps past the segment and for
  // partners before the record (loads at clamped steps, the conditions are scalar)
  auto chunk = [&](int64_t s, auto Jc) {
    constexpr int J = decltype(Jc)::value;
    float a[kEssChunk], b[kEssChunk];
    const float* p = x + (s < T ? s : T - 1) * st;
    const float* q = x + (s > lag ? s - lag : 0) * st;
#pragma unroll
    for (int j = 0; j < kEssChunk; ++j) {
      a[j] = p[cl];
      if (s + j + 1 < T) p += st;
      if constexpr (!LAG0) {
        b[j] = q[cl];
        if (s + j >= lag) q += st;  // s + j < T or unused, so q stays in the record
      }
    }
#pragma unroll
    for (int j = 0; j < kEssChunk; ++j) {
      double y = (double)a[j] - mc;
      if (s + j >= s1) y = 0.0;
      // w[slot] holds the delayed value of the latest step congruent to slot; at lag 0 that is
      // y itself (zero past the segment, where it only meets zeros)
      if constexpr (LAG0) w[J + j] = y;
      else w[J + j] = s + j >= lag ? (double)b[j] - mc : 0.0;
#pragma unroll
      for (int k = 0; k < kEssLB; ++k) acc[k] += y * w[(J + j - k + kEssLB) % kEssLB];
      __builtin_amdgcn_sched_barrier(0);  // keep the conversions from piling up in registers
    }
  };
  if (s0 < s1 && s1 > lag) {
    const int64_t u0 = s0 - kEssLB - lag;
    const float* q = x + (u0 > 0 ? u0 : 0) * st;
#pragma unroll
    for (int j = 0; j < kEssLB; ++j) {
      w[j] = u0 + j >= 0 ? (double)q[cl] - mc : 0.0;
      if (u0 + j >= 0) q += st;
    }
    for (int64_t s = s0; s < s1; s += kEssLB) {
      chunk(s, std::integral_constant<int, 0>{});
      chunk(s + kEssChunk, std::integral_constant<int, kEssChunk>{});
    }
  }
  // sum over the 64 chains: halve the sums per lane while pairing lanes
#pragma unroll
  for (int k = 0; k < kEssLB; ++k) acc[k] = valid ? acc[k] : 0.0;
#pragma unroll
  for (int n = kEssLB / 2, o = 32; n >= 1; n >>= 1, o >>= 1) {
    const bool up = lane & o;
#pragma unroll
    for (int k = 0; k < kEssLB / 2; ++k) {
      if (k < n) {
        const double send = up ? acc[k] : acc[k + n], keep = up ? acc[k + n] : acc[k];
        acc[k] = keep + __shfl_xor(send, o, 64);
      }
    }
  }
  const double r = acc[0] + __shfl_xor(acc[0], 1, 64);
  if (!(lane & 1))
    part[(((int64_t)i * gridDim.x + cb) * n_seg + sg) * (n_win * kEssLB) + win * kEssLB + (lane >> 1)] = r;
}

// out[i][l] = sum over the n partial sums of parameter i, eight interleaved runs in order
__global__ void ess_sum_kernel(const double* part, int64_t n, int n_lag, double* out) {
  __shared__ double sh[8][kEssLB];
  const int i = blockIdx.x, l = threadIdx.x % kEssLB, q = threadIdx.x / kEssLB;
  const int lag = blockIdx.y * kEssLB + l;
  const double* p = part + (int64_t)i * n * n_lag + lag;
  double s = 0;
#pragma unroll 4
  for (int64_t b = q; b < n; b += 8) s += p[b * n_lag];
  sh[q][l] = s;
  __syncthreads();
  if (q == 0) {
    s = 0;
    for (int w = 0; w < 8; ++w) s += sh[w][l];
    out[i * n_lag + lag] = s;
  }
}

// ---- fixed scratch of the entry points that allocate nothing ------------------------------
// One copy per GPU in the code object's global segment, held until the process ends.  Host
// code never passes this name to a kernel: the host-side symbol is not a device address.
// Kernels get the per-device address that noalloc_scratch_address resolved.
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
double* scratch_dev[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_address(int dev, double** p) {
  *p = nullptr;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_dev[dev]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != dev) return hipErrorInvalidDevice;  // resolved with its own device current
    void* q = nullptr;
    e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_dev[dev] = (double*)q;
  }
  *p = scratch_dev[dev];
  return hipSuccess;
}

// ---- table of the plain model's oscillations and data -----------------------------------------
// The argument (2 pi k) x as a sum of two doubles, so that cosine and sine are rounded once; zero
// rows (weight 0) past the last bin.
__global__ void plain_table_kernel(Target tg, f64x2* table) {
  const int rows = tg.n_terms + 1;
  const int64_t n = (int64_t)(tg.n_bins + 63) / 64 * 64 * rows;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e / (64 * rows) * 64 + (e & 63);
    const int m = (int)(e / 64 % rows);
    f64x2 v = {0.0, 0.0};
    if (j < tg.n_bins && m < tg.n_terms) {
      const double w = 2.0 * 3.141592653589793 * tg.pk[m], x = tg.xgrid[j];
      const double hi = w * x, lo = fma(w, x, -hi);
      double sh, ch, sl, cl;
      sincos(hi, &sh, &ch);
      sincos(lo, &sl, &cl);
      v = f64x2{ch * cl - sh * sl, sh * cl + ch * sl};
    } else if (j < tg.n_bins) {
      v = f64x2{tg.data[j], tg.w2[j]};
    }
    table[e] = v;
  }
}

// ---- batch log pi of the plain model (no gradient): NP points per wave ------------------------
// The tile kernels hold a workgroup per CU with the registers of the emulator passes, one wave per
// SIMD; here two or three share one.  Bound by the rows of plain_wave's table, 320 KB per wave for 2500
// bins x 8 terms from L2 (50 B per clock and CU), hence several points per wave, and with few points by
// the latency of its 40 dependent chunks.  The sums of the Gaussian part and of the penalty keep the
// tile kernels' component order.
template <int NP>
__global__ __launch_bounds__(64) void plain_eval_kernel(KArgs a) {
  const Target& tg = a.tg;
  const int lane = threadIdx.x, d = tg.d;
  const int64_t c0 = (int64_t)blockIdx.x * NP;
  const int mv = a.st.N - c0 < NP ? (int)(a.st.N - c0) : NP;
  const TView X{const_cast<double*>(a.ex_x) + c0, a.ex_pitch};
  int c[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) c[p] = p < mv ? p : mv - 1;
  double pl[NP];
  plain_wave<NP>(tg, X, c, pl);
  const int i = lane < d ? lane : d - 1;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (p >= mv) break;
    const double x = X(i, p);
    const bool in = __ballot(lane < d && !(x >= tg.lower[i] && x <= tg.upper[i])) == 0;
    double lp = tg.offset;
    if (tg.gauss_coef != 0.0) {
      double y = x;
      if (tg.tw_v >= 0) {
        const double du = lane_value(x, tg.tw_u) - tg.tw_center;
        if (i == tg.tw_v) y = y + tg.tw_beta * (du * du - tg.tw_kappa);
      }
      const double R = y - tg.gmean[i];
      double PR = 0, q = 0;
      for (int j = 0; j < d; ++j) PR += tg.gprec[i * d + j] * lane_value(R, j);
      for (int j = 0; j < d; ++j) q += lane_value(R, j) * lane_value(PR, j);
      lp += tg.gauss_coef * (-0.5 * q);
    }
    lp += pl[p];
    if (tg.box_penalty) {
      if (!in) {
        double dp;
        const double pen = box_pen(tg, i, x, &dp);
        for (int j = 0; j < d; ++j) lp -= lane_value(pen, j);
      }
    } else if (!in) {
      lp = -INFINITY;
    }
    if (lane == 0) a.ex_lp[c0 + p] = lp;
  }
}

// ---- layout conversion: dst[j][i] = src[i][j] for a rows x cols row-major source ----------
__global__ void transpose_kernel(const double* src, int64_t rows, int64_t cols, double* dst) {
  const int64_t total = rows * cols;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / cols, j = e % cols;
    dst[j * rows + i] = src[e];
  }
}

// ---- training inputs: t[c][i] = (x[i][c] - center[i]) invscale[i], FP64 SoA in, FP32 AoS out
__global__ void normalise_inputs_kernel(const double* x, int64_t n, int d, InputScaling sc,
                                        float* t) {
  const int64_t total = (int64_t)d * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e / d;
    const int i = (int)(e % d);
    t[e] = (float)((x[(int64_t)i * n + c] - sc.center[i]) * sc.invscale[i]);
  }
}

// ---- weight gradients: one launch for every parameter ------------------------------------
// Blocks [0, n_gemm): dW_l = delta_l h_{l-1}^T, l >= 2, on FP32 MFMA, K = batch; the blocks
// after them: dW_1, the biases, w_out and b_out as FP64 sums over the batch.
//
// GEMM blocks.  Each wave owns R x R tiles of 16 x 16 outputs and walks the whole batch, so
// every output has one accumulator whose order does not depend on R.  Both operands lie in
// fragment order (1 KiB contiguous per fragment) and are loaded kDwRing k-steps ahead: at
// R = 2 a wave loads 4 KiB per 512 MFMA cycles, 32 B per clock and CU, below what L2 delivers,
// so LDS staging would only add barriers.  The bound is the FP32 matrix rate at R = 2 and the
// serial accumulator chain (128 cycles per 16 points) at R = 1.  512 x 4 layers, 1024 points:
// 20.4 us (13.7 us of MFMA); 35 us with the operands as rows of the batch (64 bytes per row, rows
// 4 KiB apart on the same L2 channels) and the ring's loads issued together at its end.
//
// Small blocks.  One workgroup per 16 rows of delta_l (bias), of delta_1 and input component
// (W_1), of h_L (w_out) and one for b_out; the waves split the batch and their FP64 sums are
// combined in wave order.
constexpr int kDwRing = 4;

struct DwArgs {
  const float *dl, *h, *th, *up;  // deltas and activations as blocks in weight-gradient order
  int64_t ldb;
  int d, H, nh;
  double* grad;
  const int64_t* offs;  // [W1, b1, b2 .. b_nh, w_out, b_out] offsets into grad (nh + 3)
  int64_t w0, wblk;     // offset of W_2 and the distance between hidden blocks
  int n_gemm;
};

// FP64 sum over the batch of f(column tile) per row of a 16-row block: lane (q, r) of each wave
// adds its points of row r, then lanes q and the waves; valid in lanes 0 .. 15 of wave 0.
constexpr int kDwWaves = kAuxThreads / 64;
template <class F>
__device__ __forceinline__ double dw_rows(int64_t CT, double (*sh)[16], const F& f) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double s = 0;
#pragma unroll 4
  for (int64_t ct = wv; ct < CT; ct += kDwWaves) s += f(ct);
  s = sum_lane_groups(s);
  __syncthreads();
  if (lane < 16) sh[wv][lane] = s;
  __syncthreads();
  s = 0;
  for (int w = 0; w < kDwWaves; ++w) s += sh[w][lane & 15];
  return s;
}

__device__ __forceinline__ void dw_small(const DwArgs& a, int b) {
  __shared__ double sh[kDwWaves][16];
  const int lane = threadIdx.x & 63, q = lane >> 4, RT = a.H / 16;
  const int64_t CT = a.ldb / 16;
  const bool own = threadIdx.x < 16;
  const f32x4* __restrict__ up = (const f32x4*)a.up + q;
  if (b < a.nh * RT) {
    const int l = b / RT, rt = b % RT, j = rt * 16 + (lane & 15);
    const f32x4* __restrict__ x = (const f32x4*)a.dl + ((int64_t)l * CT * RT + rt) * 64 + lane;
    const double s = dw_rows(CT, sh, [&](int64_t ct) {
      const f32x4 v = x[ct * RT * 64];
      return ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
    });
    if (own) a.grad[a.offs[1 + l] + j] = s;
  } else if ((b -= a.nh * RT) < a.d * RT) {
    const int i = b / RT, rt = b % RT;
    const f32x4* __restrict__ x = (const f32x4*)a.dl + (int64_t)rt * 64 + lane;
    const f32x4* __restrict__ t = (const f32x4*)(a.th + i * a.ldb) + q;
    const double s = dw_rows(CT, sh, [&](int64_t ct) {
      const f32x4 v = x[ct * RT * 64], u = t[ct * 4];
      double p = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) p += (double)v[r] * u[r];
      return p;
    });
    if (own) a.grad[a.offs[0] + (int64_t)(rt * 16 + lane) * a.d + i] = s;
  } else if ((b -= a.d * RT) < RT) {
    const int rt = b;
    const f32x4* __restrict__ x =
        (const f32x4*)a.h + ((int64_t)(a.nh - 1) * CT * RT + rt) * 64 + lane;
    const double s = dw_rows(CT, sh, [&](int64_t ct) {
      const f32x4 v = x[ct * RT * 64], u = up[ct * 4];
      double p = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) p += (double)u[r] * v[r];
      return p;
    });
    if (own) a.grad[a.offs[1 + a.nh] + rt * 16 + lane] = s;
  } else {
    const double s = dw_rows(CT, sh, [&](int64_t ct) {
      const f32x4 u = up[ct * 4];
      return ((double)u[0] + (double)u[1]) + ((double)u[2] + (double)u[3]);
    });
    if (threadIdx.x == 0) a.grad[a.offs[2 + a.nh]] = s;
  }
}

template <int R>
__global__ __launch_bounds__(kAuxThreads) void dw_kernel(DwArgs a) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 4, cl = lane & 15;
  if ((int)blockIdx.x >= a.n_gemm) {
    dw_small(a, blockIdx.x - a.n_gemm);
    return;
  }
  constexpr int TB = 2 * R;  // block tile in 16 x 16 outputs
  const int RT = a.H / 16, nt = RT / TB, per = nt * nt;
  const int b = xcd_run(blockIdx.x, a.n_gemm);
  const int l = b / per, t = b % per;
  const int r0 = (t / nt) * TB + (wv >> 1) * R, k0 = (t % nt) * TB + (wv & 1) * R;
  const int64_t ns = a.ldb / 16;           // k-steps
  const int64_t st = (int64_t)RT * 64;     // fragments per k-step
  const f32x4* __restrict__ A = (const f32x4*)a.dl + ((l + 1) * ns * RT + r0) * 64 + lane;
  const f32x4* __restrict__ B = (const f32x4*)a.h + (l * ns * RT + k0) * 64 + lane;
  f32x4 acc[R][R] = {};
  f32x4 fa[kDwRing][R], fb[kDwRing][R];
  int64_t next = 0, o = 0;  // the k-step loaded next (the last one again past the end)
  auto load = [&](int p) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      fa[p][r] = A[r * 64 + o];
      fb[p][r] = B[r * 64 + o];
    }
    if (++next < ns) o += st;
  };
#pragma unroll
  for (int p = 0; p < kDwRing; ++p) load(p);
  auto mma = [&](int p) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[p][i][q], fb[p][j][q], acc[i][j], 0,
                                                           0, 0);
  };
  int64_t s0 = 0;
  for (; s0 + kDwRing <= ns; s0 += kDwRing) {
#pragma unroll
    for (int p = 0; p < kDwRing; ++p) {
      mma(p);
      load(p);
      __builtin_amdgcn_sched_barrier(0);  // else every load of the ring is issued at its end
    }
  }
#pragma unroll
  for (int p = 0; p < kDwRing; ++p)
    if (s0 + p < ns) mma(p);
  double* gW = a.grad + a.w0 + l * a.wblk;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        gW[(int64_t)((r0 + i) * 16 + 4 * g + r) * a.H + (k0 + j) * 16 + cl] = (double)acc[i][j][r];
}

__global__ void sum_kernel(const double* part, int n, double scale, double* out) {
  __shared__ double sh[kAuxThreads];
  double v = 0;
  for (int i = threadIdx.x; i < n; i += kAuxThreads) v += part[i];
  v = block_sum(v, sh);
  if (threadIdx.x == 0) *out = v * scale;
}

// ---- standardisation and importance weights (fixed-order two-stage reductions) ---------
// mode 0: sum a;  1: sum (a - s)^2;  2: max (a - b);  3: sum e, sum e^2 with e = exp(a - b - s)
__global__ void reduce_partial_kernel(int mode, const double* a, const double* b, int64_t n,
                                      double s, double* part) {
  __shared__ double sh[kAuxThreads];
  __shared__ double sh2[kAuxThreads];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t i0 = blockIdx.x * per, i1 = min(n, i0 + per);
  double v = mode == 2 ? -INFINITY : 0.0, v2 = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kAuxThreads) {
    if (mode == 0) v += a[i];
    else if (mode == 1) { const double r = a[i] - s; v += r * r; }
    else if (mode == 2) v = fmax(v, a[i] - b[i]);
    else { const double e = exp(a[i] - b[i] - s); v += e; v2 += e * e; }
  }
  sh[threadIdx.x] = v;
  sh2[threadIdx.x] = v2;
  __syncthreads();
  for (int k = kAuxThreads / 2; k > 0; k >>= 1) {
    if (threadIdx.x < k) {
      if (mode == 2) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + k]);
      else sh[threadIdx.x] += sh[threadIdx.x + k];
      sh2[threadIdx.x] += sh2[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = sh[0];
    part[2 * blockIdx.x + 1] = sh2[0];
  }
}

__global__ void reduce_final_kernel(int mode, const double* part, int nb, double* out) {
  if (threadIdx.x != 0) return;
  double v = mode == 2 ? -INFINITY : 0.0, v2 = 0.0;
  for (int k = 0; k < nb; ++k) {
    if (mode == 2) v = fmax(v, part[2 * k]);
    else v += part[2 * k];
    v2 += part[2 * k + 1];
  }
  out[0] = v;
  out[1] = v2;
}

__global__ void standardise_kernel(const double* y, int64_t n, const double* stats, float* out) {
  // stats = [sum, -, sum sq dev, -]: mean = sum / n, sigma = sqrt(sum sq dev / n)
  const double mu = stats[0] / (double)n, sig = sqrt(stats[2] / (double)n);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (float)((y[i] - mu) / sig);
}

__global__ void weights_kernel(const double* a, const double* b, int64_t n, const double* st,
                               double* w) {
  // st = [max, -, sum e, sum e^2]
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    w[i] = exp(a[i] - b[i] - st[0]) / st[2];
}

}  // namespace best

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
namespace best {

static int grid_for(int64_t n) {
  int64_t g = (n + kAuxThreads - 1) / kAuxThreads;
  if (g < 1) g = 1;
  if (g > 8192) g = 8192;
  return (int)g;
}

hipError_t launch_init_positions(const Target& tg, const State& S, const Rng& rng, int mode,
                                 const double* pt, double scale, const double* L0,
                                 uint64_t step, hipStream_t s) {
  hipLaunchKernelGGL(init_positions_kernel, dim3(grid_for((int64_t)tg.d * S.N)),
                     dim3(kAuxThreads), 0, s, tg, S, rng, mode, pt, scale, L0, step);
  return hipGetLastError();
}

hipError_t launch_rewhiten(const State& S, const Whiten& W, int d, hipStream_t s) {
  hipLaunchKernelGGL(rewhiten_kernel, dim3(grid_for(S.N)), dim3(kAuxThreads), 0, s, S, W, d);
  return hipGetLastError();
}

hipError_t launch_da_update(const double* step_prob, int64_t N, double* da, hipStream_t s) {
  hipLaunchKernelGGL(da_update_kernel, dim3(1), dim3(kAuxThreads), 0, s, step_prob, N, da);
  return hipGetLastError();
}

hipError_t launch_stats(const State& S, int64_t* out_i, double* out_d, hipStream_t s) {
  hipLaunchKernelGGL(stats_kernel, dim3(1), dim3(kAuxThreads), 0, s, S, out_i, out_d);
  return hipGetLastError();
}

hipError_t launch_aies_record(const State& S, int d, float* rec, int64_t slot, int64_t pitch,
                              hipStream_t s) {
  hipLaunchKernelGGL(aies_record_kernel, dim3(grid_for((int64_t)d * S.N)), dim3(kAuxThreads), 0,
                     s, S, d, rec, slot, pitch);
  return hipGetLastError();
}

hipError_t launch_moment_sums(const float* rec, const double* xs, int64_t T, int64_t N,
                              int64_t pitch, int d, const double* shift, int64_t spitch,
                              double* part, int nblocks, hipStream_t s) {
  const dim3 g(nblocks), b(64 * kMomWaves);
  const bool vec = N % 4 == 0;
#define BEST_MOMENTS(D16)                                                                        \
  if (!rec) hipLaunchKernelGGL((moments_partial_kernel<D16, false, false>), g, b, 0, s, rec, xs, \
                               T, N, pitch, d, shift, spitch, part);                             \
  else if (vec) hipLaunchKernelGGL((moments_partial_kernel<D16, true, true>), g, b, 0, s, rec,   \
                                   xs, T, N, pitch, d, shift, spitch, part);                     \
  else hipLaunchKernelGGL((moments_partial_kernel<D16, true, false>), g, b, 0, s, rec, xs, T, N, \
                          pitch, d, shift, spitch, part)
  if (d <= 16) {
    BEST_MOMENTS(1);
  } else {
    BEST_MOMENTS(2);
  }
#undef BEST_MOMENTS
  return hipGetLastError();
}

hipError_t launch_moments(const float* rec, const double* xs, int64_t T, int64_t N,
                          int64_t pitch, int d, const double* shift, double* part, int nblocks,
                          int update_mean, double* mu, double* L, double* info, hipStream_t s) {
  hipLaunchKernelGGL(adapt_moments_kernel, dim3(nblocks), dim3(kAuxThreads), 0, s, rec, xs, T, N,
                     pitch, d, shift, part);
  hipLaunchKernelGGL(moments_final_kernel, dim3(1), dim3(kAuxThreads), 0, s, part, nblocks,
                     T * N, d, shift, update_mean, mu, L, info);
  return hipGetLastError();
}

hipError_t launch_ess_chain_stats(const float* rec, int64_t T, int d, int64_t N, double* mean,
                                  double* ssq, hipStream_t s) {
  const int64_t hi = (T + kStatWaves - 1) / kStatWaves, lo = hi - 1;
  auto inv = [](int64_t n) { return n ? 1.0 / (double)n : 0.0; };
  const StatSteps n{(int)(T - lo * kStatWaves), (double)hi, (double)lo, 1.0 / (double)T, inv(hi), inv(lo),
                    inv(hi % kStatBlock), inv(lo % kStatBlock)};
  hipLaunchKernelGGL(ess_chain_stats_kernel,
                     dim3((unsigned)capped_blocks((N + 63) / 64, 64 * kStatWaves), (unsigned)d),
                     dim3(64 * kStatWaves), 0, s, rec, T, d, N, n, mean, ssq);
  return hipGetLastError();
}

hipError_t launch_ess_param_stats(const double* mean, const double* ssq, int64_t N, int d,
                                  double* out, hipStream_t s) {
  hipLaunchKernelGGL(ess_param_stats_kernel, dim3((unsigned)d), dim3(kAuxThreads), 0, s, mean, ssq,
                     N, out);
  return hipGetLastError();
}

hipError_t launch_ess_autocov(const float* rec, const double* mean, int64_t T, int d, int64_t N,
                              int64_t lag0, int n_win, int n_seg, double* part, double* out,
                              hipStream_t s) {
  const int64_t nblk = (N + 63) / 64;
  const int64_t seg = ((T + n_seg - 1) / n_seg + kEssLB - 1) / kEssLB * kEssLB;
  const dim3 grid((unsigned)nblk, (unsigned)d, (unsigned)(n_seg * n_win));
  if (lag0 == 0)
    hipLaunchKernelGGL((ess_autocov_kernel<true>), grid, dim3(64), 0, s, rec, mean, T, d, N, lag0,
                       1, seg, part);
  else
    hipLaunchKernelGGL((ess_autocov_kernel<false>), grid, dim3(64), 0, s, rec, mean, T, d, N, lag0,
                       n_win, seg, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ess_sum_kernel, dim3((unsigned)d, (unsigned)n_win), dim3(8 * kEssLB), 0, s, part,
                     nblk * n_seg, n_win * kEssLB, out);
  return hipGetLastError();
}

hipError_t launch_plain_table(const Target& tg, f64x2* table, hipStream_t s) {
  hipLaunchKernelGGL(plain_table_kernel, dim3(grid_for((int64_t)(tg.n_bins + 63) / 64 * 64 * (tg.n_terms + 1))),
                     dim3(kAuxThreads), 0, s, tg, table);
  return hipGetLastError();
}

// Points per wave: one while the chip's SIMDs (n_cu x 4) get no more than a wave each, then as many as
// two waves per SIMD hold at once, at most three (us for 1000 / 2048 / 4096 / 6000 / 20000 points: one
// per wave 17.2 / 28.1 / 49.3 / 69.8 / 224, two 20.5 / 21.3 / 32.9 / 46.4 / 134, three 25.9 / 26.0 / 37.2 /
// 38.7 / 120; four need more registers than two waves have).  Without the table there is nothing to share.
// A grid has fewer than 2^32 work items: larger batches are split here (a loop over the points in the
// kernel keeps 50 registers more alive, one wave per SIMD fewer).
hipError_t launch_plain_eval(const KArgs& a, int n_cu, hipStream_t s) {
  const int64_t n = a.st.N;
  const int np = n <= 4 * n_cu || !a.tg.pl_even ? 1 : n <= 16 * n_cu ? 2 : 3;
  KArgs k = a;
  for (int64_t c = 0; c < n;) {
    const int64_t blocks = capped_blocks((n - c + np - 1) / np, 64);
    k.st.N = n - c < blocks * np ? n - c : blocks * np;
    k.ex_x = a.ex_x + c;
    k.ex_lp = a.ex_lp + c;
    const dim3 g((unsigned)blocks), b(64);
    if (np == 1) hipLaunchKernelGGL((plain_eval_kernel<1>), g, b, 0, s, k);
    else if (np == 2) hipLaunchKernelGGL((plain_eval_kernel<2>), g, b, 0, s, k);
    else hipLaunchKernelGGL((plain_eval_kernel<3>), g, b, 0, s, k);
    if (hipError_t e = hipGetLastError()) return e;
    c += k.st.N;
  }
  return hipSuccess;
}

hipError_t launch_transpose(const double* src, int64_t rows, int64_t cols, double* dst,
                            hipStream_t s) {
  hipLaunchKernelGGL(transpose_kernel, dim3(grid_for(rows * cols)), dim3(kAuxThreads), 0, s, src,
                     rows, cols, dst);
  return hipGetLastError();
}

hipError_t launch_normalise_inputs(const double* x, int64_t n, int d, const InputScaling& sc,
                                   float* t, hipStream_t s) {
  hipLaunchKernelGGL(normalise_inputs_kernel, dim3(grid_for((int64_t)d * n)), dim3(kAuxThreads),
                     0, s, x, n, d, sc, t);
  return hipGetLastError();
}

hipError_t launch_dw(const FitArgs& f, double* grad, const int64_t* offs, hipStream_t s) {
  const int d = f.mp.d, H = f.mp.H, nh = f.mp.nh;
  DwArgs a{f.act, f.hx, f.th, f.up, f.ldb, d, H, nh, grad, offs, (int64_t)H * d + H,
           (int64_t)H * H + H, 0};
  const int64_t small = (int64_t)(nh + d + 1) * (H / 16) + 1;
  // 2 x 2 tiles per wave once that still gives half of the chip's 1024 SIMDs a wave (each
  // operand load then serves two MFMAs; 512 x 4 layers: 768 waves); below, one tile per wave,
  // which four times as many SIMDs share (128 x 2 and 1024 points: 16 waves against 64)
  const int64_t tiles = (int64_t)(nh - 1) * (H / 16) * (H / 16);
  if (tiles / 4 >= 512) {
    a.n_gemm = (int)(tiles / 16);
    // GEMM blocks that do not fill the 256 CUs ask for more than half of a CU's LDS: one block
    // per CU, so the small blocks run on the other CUs instead of beside GEMM waves (512 x 4
    // layers, 1024 points: 20.4 us against 24.7)
    const size_t lds = a.n_gemm <= 256 ? 84 * 1024 : 0;
    hipError_t e = hipFuncSetAttribute((const void*)dw_kernel<2>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 84 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((dw_kernel<2>), dim3((unsigned)(a.n_gemm + small)), dim3(kAuxThreads), lds, s, a);
  } else {
    a.n_gemm = (int)(tiles / 4);
    hipLaunchKernelGGL((dw_kernel<1>), dim3((unsigned)(a.n_gemm + small)), dim3(kAuxThreads), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_sum(const double* part, int n, double scale, double* out, hipStream_t s) {
  hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(kAuxThreads), 0, s, part, n, scale, out);
  return hipGetLastError();
}


static hipError_t reduce2(int mode, const double* a, const double* b, int64_t n, double shift,
                          double* part, double* out, hipStream_t s) {
  const int nb = 256;
  hipLaunchKernelGGL(reduce_partial_kernel, dim3(nb), dim3(kAuxThreads), 0, s, mode, a, b, n,
                     shift, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(64), 0, s, mode, part, nb, out);
  return hipGetLastError();
}

// scratch: >= 512 + 4 doubles of device memory
hipError_t launch_standardise(const double* y, int64_t n, float* out, double* scratch,
                              double* stats_host, hipStream_t s) {
  double* part = scratch;
  double* st = scratch + 512;
  hipError_t e = reduce2(0, y, nullptr, n, 0.0, part, st, s);
  if (e != hipSuccess) return e;
  double sum[2];
  if ((e = hipMemcpyAsync(sum, st, 16, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  const double mu = sum[0] / (double)n;
  if ((e = reduce2(1, y, nullptr, n, mu, part, st + 2, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(standardise_kernel, dim3(grid_for(n)), dim3(kAuxThreads), 0, s, y, n, st, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(stats_host, st, 32, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

hipError_t launch_importance_weights(const double* lp, const double* le, int64_t n, double* w,
                                     double* scratch, double* stats_host, hipStream_t s) {
  double* part = scratch;
  double* st = scratch + 512;
  hipError_t e = reduce2(2, lp, le, n, 0.0, part, st, s);
  if (e != hipSuccess) return e;
  double mx[2];
  if ((e = hipMemcpyAsync(mx, st, 16, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  if ((e = reduce2(3, lp, le, n, mx[0], part, st + 2, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(weights_kernel, dim3(grid_for(n)), dim3(kAuxThreads), 0, s, lp, le, n, st, w);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(stats_host, st, 32, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

}  // namespace best
