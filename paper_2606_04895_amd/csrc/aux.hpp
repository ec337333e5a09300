// Host-visible launchers of the library's kernels.  Each is defined in the translation
// unit that defines the kernel it launches.
#pragma once
#include "train.hpp"
#include "launch.hpp"

namespace best {

constexpr int kEssLB = 32;   // lags per autocovariance window
constexpr int kEssWin = 4;   // windows per launch after the first launch's single one
// Partial sums of an autocovariance launch where a single time segment fits in that many.
constexpr int64_t kEssPartials = (int64_t)1 << 21;
// Time segments of the autocovariance launches: enough that 4096 waves (four per SIMD) share
// the record, none shorter than 128 steps, and the partial sums of kEssWin windows no more than
// kEssPartials doubles where one segment fits in that (every size best_ess_noalloc takes).
inline int ess_segments(int64_t T, int d, int64_t N) {
  const int64_t rows = (int64_t)d * ((N + 63) / 64);
  int64_t n = (4096 + rows - 1) / rows;
  if (n > T / 128) n = T / 128;
  const int64_t cap = kEssPartials / (rows * kEssWin * kEssLB);
  if (n > cap) n = cap;
  return (int)(n < 1 ? 1 : n);
}
// Entry points that allocate nothing take their device scratch from one fixed array per
// GPU (kernels_aux.hip).  The ESS passes need the means and sums of squares, 2 d N doubles, and up
// to kEssPartials partial sums, so d times the 64-padded chain count is limited to kNoAllocMaxDN (32 MiB
// of scratch per GPU).
constexpr int64_t kNoAllocMaxDN = (int64_t)1 << 20;
constexpr int64_t kNoAllocScratchDoubles = 4 * kNoAllocMaxDN;
static_assert(kNoAllocScratchDoubles >= 2 * kNoAllocMaxDN + kEssPartials &&
                  kNoAllocMaxDN / 64 * kEssWin * kEssLB <= kEssPartials,
              "fixed scratch: means, squares and one segment's partial sums of the largest record");

// Templated per precision (kernels_<prec>.hip).
hipError_t launch_step(int prec, int MT, const KArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_eval(int prec, int MT, const KArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_pack(int prec, const double* flat, int d, int H, int nh, void* wf, void* wb,
                       void* w1f, void* w1t, void* bias, void* wout, hipStream_t s);
hipError_t launch_fit(int prec, const FitArgs& a, hipStream_t s);
hipError_t launch_eval_layers(int prec, const KArgs& k, const FitArgs& f, size_t lds, hipStream_t s);
hipError_t launch_adam_pack(int prec, const AdamArgs& a, hipStream_t s);

// kernels_aux.hip
hipError_t launch_init_positions(const Target& tg, const State& S, const Rng& rng, int mode,
                                 const double* pt, double scale, const double* L0,
                                 uint64_t step, hipStream_t s);
hipError_t launch_rewhiten(const State& S, const Whiten& W, int d, hipStream_t s);
hipError_t launch_da_update(const double* step_prob, int64_t N, double* da, hipStream_t s);
hipError_t launch_stats(const State& S, int64_t* out_i, double* out_d, hipStream_t s);
hipError_t launch_aies_record(const State& S, int d, float* rec, int64_t slot, int64_t pitch,
                              hipStream_t s);
hipError_t launch_moments(const float* rec, const double* xs, int64_t T, int64_t N,
                          int64_t pitch, int d, const double* shift, double* part, int nblocks,
                          int update_mean, double* mu, double* L, double* info, hipStream_t s);
hipError_t launch_moment_sums(const float* rec, const double* xs, int64_t T, int64_t N,
                              int64_t pitch, int d, const double* shift, int64_t spitch,
                              double* part, int nblocks, hipStream_t s);
hipError_t launch_ess_chain_stats(const float* rec, int64_t T, int d, int64_t N, double* mean,
                                  double* ssq, hipStream_t s);
// Device address of GPU dev's copy of the fixed scratch array (kNoAllocScratchDoubles
// doubles).  The first call for a device must have that device current; the address is
// kept per device and later calls return it.
hipError_t noalloc_scratch_address(int dev, double** p);
hipError_t launch_ess_param_stats(const double* mean, const double* ssq, int64_t N, int d,
                                  double* out, hipStream_t s);
hipError_t launch_ess_autocov(const float* rec, const double* mean, int64_t T, int d, int64_t N,
                              int64_t lag0, int n_win, int n_seg, double* part, double* out,
                              hipStream_t s);
// the rows that plain_bin reads: cos, sin of (2 pi k_m) x_j and (data, weight) of every bin
hipError_t launch_plain_table(const Target& tg, f64x2* table, hipStream_t s);
// log pi of a.st.N points a.ex_x into a.ex_lp, plain model alone (plain_mode 2)
hipError_t launch_plain_eval(const KArgs& a, int n_cu, hipStream_t s);
hipError_t launch_transpose(const double* src, int64_t rows, int64_t cols, double* dst,
                            hipStream_t s);
struct InputScaling {  // kernel argument: per-component centre and inverse scale
  double center[kMaxD], invscale[kMaxD];
};
hipError_t launch_normalise_inputs(const double* x, int64_t n, int d, const InputScaling& sc,
                                   float* t, hipStream_t s);
hipError_t launch_dw(const FitArgs& a, double* grad, const int64_t* offs, hipStream_t s);
hipError_t launch_sum(const double* part, int n, double scale, double* out, hipStream_t s);
hipError_t launch_standardise(const double* y, int64_t n, float* out, double* scratch,
                              double* stats_host, hipStream_t s);
hipError_t launch_importance_weights(const double* lp, const double* le, int64_t n, double* w,
                                     double* scratch, double* stats_host, hipStream_t s);

// metrics.hip (convergence metrics of Sec. 4.1)
hipError_t launch_whiten_points(const float* rec, int64_t T, int d, int64_t N, const double* mu,
                                const double* L, double* z, int64_t zpitch, hipStream_t s);
hipError_t launch_sum_parts(const double* part, int nblocks, int np, double* out, hipStream_t s);
hipError_t launch_directions(const Rng& rng, int d, int K, double* w, hipStream_t s);
// W1 of P projections (w [P][d]) of the points za ([d][na]) and zb ([d][nb]) into out[P]; keys and
// tmp: P (na + nb) words, part: P sliced_w1_parts(na + nb) doubles.
int64_t sliced_w1_parts(int64_t n);
hipError_t launch_sliced_w1(const double* za, int64_t na, const double* zb, int64_t nb, int d,
                            const double* w, int P, uint64_t* keys, uint64_t* tmp, double* part,
                            double* out, hipStream_t s);
// Four order statistics of every row of z [d][n] (synchronises).
size_t select_scratch_bytes(int d);
hipError_t select_ranks(const double* z, int d, int64_t n, const int64_t* ranks, void* scratch,
                        double* out, hipStream_t s);

}  // namespace best
