// Templated kernels for weight packing and for the passes that need weight gradients (emulator
// training and the vector-Jacobian product of the target): layer-by-layer forward and reverse
// passes over a batch that leave every activation and delta in the weight-gradient GEMMs'
// operand order.
#pragma once
#include "kernels.hpp"

namespace best {

// Flat FP64 parameters -> packed device copies used by the tile engine:
//   wf: W_l in fragment order (rows = outputs), wb: W_l^T in fragment order (l >= 2),
//   w1f: W_1 in the input layer's fragment order (k = input component, zero padded),
//   w1t: W_1^T in fragment order (rows = input components, zero padded to 16 rti),
//   bias: [nh][H], wout: [H] followed by b_out.
// Rounding of a parameter to a storage type: to nearest, in one step (written as two conversions
// through FP32, the compiler folds them for 16-bit types in some places and not in others, which
// differ on ties).
template <class T>
__device__ __forceinline__ T to_store(double v) {
  return (T)v;
}

template <class P>
__global__ void pack_kernel(const double* flat, int d, int H, int nh, typename P::T* wf,
                            typename P::T* wb, void* w1f_, typename P::T* w1t,
                            typename P::acc* bias, typename P::acc* wout) {
  using T = typename P::T;
  using IP = typename InPrec<P>::type;
  typename IP::T* w1f = (typename IP::T*)w1f_;
  const int64_t HH = (int64_t)H * H;
  const int64_t nW = (int64_t)(nh - 1) * HH;
  const int64_t ks1 = (d + IP::KSTEP - 1) / IP::KSTEP, K1 = ks1 * IP::KSTEP;
  const int64_t R1 = (d + 15) / 16 * 16;
  const int64_t n1f = (int64_t)H * K1, n1t = R1 * H;
  const int64_t total = nW + n1f + n1t + (int64_t)nh * H + H + 1;
  const int64_t KS = H / P::KSTEP;
  const int64_t offb1 = (int64_t)H * d;
  const int64_t blk = HH + H;  // one hidden block W_l + b_l (l >= 2)
  const int64_t offwo = offb1 + H + (int64_t)(nh - 1) * blk;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (e < nW) {
      const int64_t l = e / HH, q = e % HH, j = q / H, k = q % H;  // layer l + 2
      const double v = flat[offb1 + H + l * blk + j * H + k];
      wf[l * HH + frag_offset<P>(j, k, KS)] = to_store<T>(v);
      wb[l * HH + frag_offset<P>(k, j, KS)] = to_store<T>(v);
    } else if (e < nW + n1f) {
      const int64_t q = e - nW, j = q / K1, i = q % K1;
      w1f[frag_offset<IP>(j, i, ks1)] = to_store<typename IP::T>(i < d ? flat[j * d + i] : 0.0);
    } else if (e < nW + n1f + n1t) {
      const int64_t q = e - nW - n1f, i = q / H, j = q % H;
      w1t[frag_offset<P>(i, j, KS)] = to_store<T>(i < d ? flat[j * d + i] : 0.0);
    } else if (e < nW + n1f + n1t + (int64_t)nh * H) {
      const int64_t q = e - nW - n1f - n1t, l = q / H, j = q % H;
      const int64_t off = l == 0 ? offb1 : offb1 + H + (l - 1) * blk + HH;
      bias[q] = (typename P::acc)flat[off + j];
    } else {
      const int64_t j = e - nW - n1f - n1t - (int64_t)nh * H;
      wout[j] = (typename P::acc)flat[offwo + j];  // j == H is b_out
    }
  }
}

// Adam on the FP64 master parameters, the packed copies of the updated parameters and the mean of
// the minibatch's loss, in one launch.  Bound by the 56 bytes per parameter of the update (44 MB for
// 512 x 4 layers, 8.7 us at the rate of a large copy; the arrays stay in the last-level cache).  A
// thread owns 4 x 4 weights of a hidden layer, so both packed orders (rows and transposed) are
// written as whole vectors from registers: 12 us for the launch, against 10 + 9 + 4.5 us as update,
// packing (which read the parameters back and scattered single elements) and loss sum.
struct AdamArgs {
  double *p, *m, *v;
  const double* g;
  double lr, b1, b2, eps, c1, c2;
  int d, H, nh;
  void *wf, *wb, *w1f, *w1t, *bias, *wout;
  const double* loss_part;
  int n_loss;
  double loss_scale;
  double* loss;
};

__device__ __forceinline__ double adam_value(const AdamArgs& a, double p, double& m, double& v,
                                             double g) {
  m = a.b1 * m + (1.0 - a.b1) * g;
  v = a.b2 * v + (1.0 - a.b2) * g * g;
  const double mh = m / a.c1, vh = v / a.c2;
  return p - a.lr * mh / (sqrt(vh) + a.eps);
}

__device__ __forceinline__ double adam_update(const AdamArgs& a, int64_t e) {
  double m = a.m[e], v = a.v[e];
  const double p = adam_value(a, a.p[e], m, v, a.g[e]);
  a.m[e] = m;
  a.v[e] = v;
  a.p[e] = p;
  return p;
}

constexpr int kAdamTile = 16 * 64;  // weights of one wave: 16 rows x 64 columns

template <class P>
__global__ __launch_bounds__(256) void adam_pack_kernel(AdamArgs a, int n_hidden_blocks) {
  using T = typename P::T;
  using IP = typename InPrec<P>::type;
  typedef T t4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int H = a.H, KS = H / P::KSTEP;
  const int64_t base = (int64_t)H * a.d + H, HH = (int64_t)H * H, blk = HH + H;
  int b = blockIdx.x;
  if (b < n_hidden_blocks) {
    const int64_t w = (int64_t)b * 4 + (tid >> 6), per = HH / kAdamTile;
    const int l = (int)(w / per), t = (int)(w % per);
    const int j0 = (t / (H / 64)) * 16 + (lane >> 4) * 4, k0 = (t % (H / 64)) * 64 + (lane & 15) * 4;
    T v[4][4];
    double* __restrict__ P0 = a.p;
    double* __restrict__ M0 = a.m;
    double* __restrict__ V0 = a.v;
    const double* __restrict__ G0 = a.g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t e = base + l * blk + (int64_t)(j0 + j) * H + k0;
      f64x2 p[2], m[2], s[2], g[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        p[u] = *(const f64x2*)(P0 + e + 2 * u);
        m[u] = *(const f64x2*)(M0 + e + 2 * u);
        s[u] = *(const f64x2*)(V0 + e + 2 * u);
        g[u] = *(const f64x2*)(G0 + e + 2 * u);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        double mk = m[k / 2][k % 2], sk = s[k / 2][k % 2];
        const double pk = adam_value(a, p[k / 2][k % 2], mk, sk, g[k / 2][k % 2]);
        m[k / 2][k % 2] = mk;
        s[k / 2][k % 2] = sk;
        p[k / 2][k % 2] = pk;
        v[j][k] = to_store<T>(pk);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        *(f64x2*)(P0 + e + 2 * u) = p[u];
        *(f64x2*)(M0 + e + 2 * u) = m[u];
        *(f64x2*)(V0 + e + 2 * u) = s[u];
      }
    }
    T* wf = (T*)a.wf + l * HH;
    T* wb = (T*)a.wb + l * HH;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      *(t4*)(wf + frag_offset<P>(j0 + j, k0, KS)) = t4{v[j][0], v[j][1], v[j][2], v[j][3]};
      *(t4*)(wb + frag_offset<P>(k0 + j, j0, KS)) = t4{v[0][j], v[1][j], v[2][j], v[3][j]};
    }
    return;
  }
  b -= n_hidden_blocks;
  // W_1, the biases, w_out and b_out, element by element
  const int64_t n1 = (int64_t)H * a.d, nb = (int64_t)a.nh * H, n = n1 + nb + H + 1;
  const int64_t q = (int64_t)b * 256 + tid;
  if (b == (n + 255) / 256) {
    // the last block: mean loss, summed in a fixed order
    __shared__ double sh[256];
    double s = 0;
    for (int i = tid; i < a.n_loss; i += 256) s += a.loss_part[i];
    sh[tid] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (tid < o) sh[tid] += sh[tid + o];
      __syncthreads();
    }
    if (tid == 0) *a.loss = sh[0] * a.loss_scale;
    return;
  }
  if (q >= n) return;
  if (q < n1) {
    const int64_t j = q / a.d, i = q % a.d, ks1 = (a.d + IP::KSTEP - 1) / IP::KSTEP;
    const double v = adam_update(a, q);
    ((typename IP::T*)a.w1f)[frag_offset<IP>(j, i, ks1)] = to_store<typename IP::T>(v);
    ((T*)a.w1t)[frag_offset<P>(i, j, KS)] = to_store<T>(v);
  } else if (q < n1 + nb) {
    const int64_t l = (q - n1) / H, j = (q - n1) % H;
    const int64_t e = l == 0 ? n1 + j : base + (l - 1) * blk + HH + j;
    ((typename P::acc*)a.bias)[q - n1] = (typename P::acc)adam_update(a, e);
  } else {
    const int64_t j = q - n1 - nb;  // j == H is b_out
    ((typename P::acc*)a.wout)[j] = (typename P::acc)adam_update(a, base + (a.nh - 1) * blk + j);
  }
}

// ---------------------------------------------------------------------------------------
// Forward and reverse pass over a batch, one launch per layer.
//
// A tile that goes through all layers in one workgroup (the samplers' form) leaves most of the
// chip idle on a minibatch: 1024 points are 64 tiles of 16.  Here each layer is a GEMM over the
// whole batch whose 16 x 16 output tiles are spread over the chip (2048 tiles for 512 x 1024),
// and a layer costs about one kernel (FP32, 512 x 512 x 1024: 7 us, of which 3.4 us are MFMA and
// the rest launch, first-touch latency and epilogue).  512 x 4 layers: the passes of a training
// step of 1024 points in FP32 took 272 us as one launch of 32-point tiles and take 56 us here;
// 4099 points in FP16 153 us and 83 us.
//
// Buffers are in units of 16 x 16 blocks (row tile rt, column tile ct = 16 points), block
// (layer, ct, rt) at ((layer * CT + ct) * RT + rt) * 256 floats:
//   act  h_l in D-slot order (lane (g, c): rows 4g .. 4g + 3 of point c), which for FP32 is also
//        the B operand of the next layer.  Each block is overwritten by delta_l (in the order of
//        hx) by the wave that read it last, so the two share the memory.
//   hx   h_l in the weight-gradient order: lane (q, r) holds points 4q .. 4q + 3 of row r.
//   pp   two panels [CT][16 H] of the GEMM type in B-fragment order: the 16-bit activations of
//        the layer just computed in the forward pass, the deltas in the reverse pass.  A batch goes
//        through the layers kFitPanel points at a time (columns are independent), which bounds them.
// Every output keeps the accumulation order of the tile engine (one accumulator per output,
// k-steps ascending), and the sums over the output weights its wave order, so the results are
// those of the tile engine bit for bit.
// ---------------------------------------------------------------------------------------
constexpr int64_t kFitPanel = 65536;
struct FitArgs {
  MlpParams mp;
  int64_t n, ldb;   // points of this pass; of the batch, rounded up to whole column tiles (strides)
  int64_t n_batch;  // points of the batch
  int round_h;      // the reverse pass takes h_l rounded to the GEMM type
  // training minibatch: rows perm[batch0 ..] of t_in [.][d] with targets y
  const float *t_in, *y;
  const int32_t* perm;
  int64_t batch0;
  double* loss_part;  // [CT] sums of squared residuals
  // target points x [d][n] (t_in == nullptr): upstream weights (NULL: ones) times mlp_coef, zero
  // for points whose log pi does not use the network
  Target tg;
  const double *x, *upstream;
  int64_t x_pitch;
  float *act, *hx;  // [nh] blocks
  float *th, *up;   // [d][ldb], [ldb]
  void *pp0, *pp1, *pp2;  // pp2: delta_{nh-1} of an evaluation, written while pp0 may be read
};

// Launch index -> tile index such that the blocks of one XCD (index mod 8) own a contiguous run
// of tiles, whose shared operands then stay in that XCD's L2.
__device__ __forceinline__ int xcd_run(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

// Transpose of the 4 x 4 blocks (4 consecutive lanes x 4 values): in lane i of a quad, v[j]
// becomes the former v[i] of lane j.
__device__ __forceinline__ float quad_xor(float v, bool by2) {
  const int b = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, by2 ? __builtin_amdgcn_mov_dpp(b, 0x4E, 0xF, 0xF, true)
                                       : __builtin_amdgcn_mov_dpp(b, 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ f32x4 quad_transpose(f32x4 v, int lane) {
  const bool o1 = lane & 1, o2 = lane & 2;
  const float a = quad_xor(o1 ? v[0] : v[1], false), b = quad_xor(o1 ? v[2] : v[3], false);
  const f32x4 w = {o1 ? a : v[0], o1 ? v[1] : a, o1 ? b : v[2], o1 ? v[3] : b};
  const float c = quad_xor(o2 ? w[0] : w[2], true), e = quad_xor(o2 ? w[1] : w[3], true);
  return f32x4{o2 ? c : w[0], o2 ? e : w[1], o2 ? w[2] : c, o2 ? w[3] : e};
}

// Slot of a D-order lane's transposed values in the weight-gradient order.
__device__ __forceinline__ int dw_slot(int lane) {
  return ((lane & 15) >> 2) * 16 + (lane >> 4) * 4 + (lane & 3);
}

__device__ __forceinline__ int64_t fit_block(const FitArgs& a, int l, int64_t ct, int rt) {
  return (((int64_t)l * (a.ldb >> 4) + ct) * (a.mp.H >> 4) + rt) * 64;
}

// The four rows of a D-slot as one column-tile panel entry of the GEMM type.  The values are
// rounded to FP32 first: folded into one instruction, the FP16 conversion of 1 - 2 rcp(..) would
// skip that rounding and differ from the tile engine's activations on ties.
template <class P>
__device__ __forceinline__ void panel_store(const FitArgs& a, typename P::T* panel, int64_t ct,
                                            int rt, int lane, f32x4 v) {
  typedef typename P::T t4 __attribute__((ext_vector_type(4)));
  using T = typename P::T;
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float f = v[r];
      asm volatile("" : "+v"(f));
      v[r] = f;
    }
  }
  const int64_t o = lds_off<P>(rt * 16 + 4 * (lane >> 4), lane & 15, a.mp.H / P::KSTEP);
  *(t4*)(panel + ct * 16 * a.mp.H + o) = t4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
}

// Input layer, kInRows row tiles of one column tile per wave (bound by latency: d <= 32).
// EVAL: for the evaluation of points, which needs no inputs or activations in the weight gradients'
// order.
constexpr int kInRows = 2;
template <class P, bool EVAL>
__global__ __launch_bounds__(256) void fit_input_kernel(FitArgs a) {
  using IP = Prec<float>;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 4, cl = lane & 15;
  const int d = a.mp.d, ks1 = a.mp.ks1;
  const int64_t ct = blockIdx.x, c = ct * 16 + cl;
  const bool valid = c < a.n;
  const bool lead = blockIdx.y == 0 && wv == 0;
  const int64_t src = valid ? (a.t_in ? (int64_t)a.perm[a.batch0 + c] : c) : 0;
  f32x4 b[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = ks * 16 + 4 * g + r;
      float v = 0.f;
      if (valid && i < d)
        v = a.t_in ? a.t_in[src * d + i]
                   : (float)((a.x[i * a.x_pitch + c] - a.tg.in_center[i]) * a.tg.in_invscale[i]);
      b[ks][r] = v;
      if (!EVAL && lead && i < d) a.th[(int64_t)i * a.ldb + c] = v;
    }
  const f32x4* __restrict__ W = (const f32x4*)a.mp.w1f + lane;
  const float* __restrict__ bias = (const float*)a.mp.bias;
#pragma unroll
  for (int rr = 0; rr < kInRows; ++rr) {
    const int rt = (blockIdx.y * 4 + wv) * kInRows + rr;
    const f32x4 bi = *(const f32x4*)(bias + rt * 16 + 4 * g);
    f32x4 v = {};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      if (ks < ks1) v = IP::mma(W[((int64_t)rt * ks1 + ks) * 64], b[ks], v);
    f32x4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = act_tanh(v[r] + bi[r]);
    const int64_t o = fit_block(a, 0, ct, rt);
    ((f32x4*)a.act)[o + lane] = h;
    if constexpr (!EVAL) ((f32x4*)a.hx)[o + dw_slot(lane)] = quad_transpose(h, lane);
    if constexpr (sizeof(typename P::T) == 2)
      if (a.mp.nh > 1) panel_store<P>(a, (typename P::T*)a.pp0, ct, rt, lane, h);
  }
}

// Hidden layer l (1 <= l < nh, activations counted from 0): forward h_l from h_{l-1}, or with
// BWD delta_{l-1} from delta_l.  R x C blocks per wave, four waves down the rows of a workgroup; the
// weights (1 KiB contiguous per fragment) and the panel fragments of the next kFitRing k-steps
// are in flight.  With C = 2 and R = 1 (the 1024-wave split of 1024 points) a wave loads
// 3 KiB per 256 FP32 MFMA cycles, 48 B per clock and CU with the panel shared through L1.
// EVAL (points, upstream 1): the last forward layer also writes delta_{nh-1} = w_out (1 - h^2), and
// every reverse layer only its panel.
constexpr int kFitRing = 4;
template <class P, int R, int C, bool BWD, bool EVAL>
__global__ __launch_bounds__(256) void fit_layer_kernel(FitArgs a, int l) {
  using T = typename P::T;
  using frag = typename P::frag;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 4;
  const int H = a.mp.H, KS = H / P::KSTEP, RT = H / 16, nrow = RT / (4 * R);
  const int64_t CT = (a.n + 15) >> 4;
  const int t = xcd_run(blockIdx.x, gridDim.x);
  const int rt0 = ((t % nrow) * 4 + wv) * R;
  const int64_t ct0 = (int64_t)(t / nrow) * C;
  const T* Aw = (const T*)(BWD ? a.mp.wb : a.mp.wf) + (int64_t)(l - 1) * H * H;
  const frag* __restrict__ A = (const frag*)Aw + (int64_t)rt0 * KS * 64 + lane;
  const int par = (a.mp.nh - 1 - l) & 1;  // reverse pass: delta_{nh-1} is in pp0
  const T* Bin;
  if constexpr (BWD) Bin = (const T*)(EVAL && l == a.mp.nh - 1 ? a.pp2 : par ? a.pp1 : a.pp0);
  else if constexpr (sizeof(T) == 4) Bin = (const T*)a.act + (l - 1) * a.ldb * H;
  else Bin = (const T*)((l & 1) ? a.pp0 : a.pp1);
  const frag* __restrict__ B[C];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int64_t ct = ct0 + j < CT ? ct0 + j : CT - 1;  // past the end: computed, not stored
    B[j] = (const frag*)Bin + ct * KS * 64 + lane;
  }
  frag fa[kFitRing][R], fb[kFitRing][C];
  auto load = [&](int p, int ks) {
#pragma unroll
    for (int i = 0; i < R; ++i) fa[p][i] = A[((int64_t)i * KS + ks) * 64];
#pragma unroll
    for (int j = 0; j < C; ++j) fb[p][j] = B[j][(int64_t)ks * 64];
  };
#pragma unroll
  for (int p = 0; p < kFitRing; ++p) load(p, p);
  f32x4 e[R][BWD ? C : 1];  // epilogue operands: bias, or the saved activations
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if constexpr (BWD) {
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const int64_t ct = ct0 + j < CT ? ct0 + j : CT - 1;
        e[i][j] = ((const f32x4*)a.act)[fit_block(a, l - 1, ct, rt0 + i) + lane];
      }
    } else {
      e[i][0] = *(const f32x4*)((const float*)a.mp.bias + (int64_t)l * H + (rt0 + i) * 16 + 4 * g);
    }
  }
  const bool last = EVAL && !BWD && l == a.mp.nh - 1;
  f32x4 wo[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if constexpr (EVAL && !BWD)
      if (last) wo[i] = *(const f32x4*)((const float*)a.mp.wout + (rt0 + i) * 16 + 4 * g);
  }
  f32x4 acc[R][C] = {};
  auto mma = [&](int p) {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < C; ++j) acc[i][j] = P::mma(fa[p][i], fb[p][j], acc[i][j]);
  };
  int k0 = 0;
  for (; k0 < KS - kFitRing; k0 += kFitRing) {
#pragma unroll
    for (int p = 0; p < kFitRing; ++p) {
      mma(p);
      load(p, k0 + p + kFitRing);
      __builtin_amdgcn_sched_barrier(0);  // else every load of the ring is issued at its end
    }
  }
#pragma unroll
  for (int p = 0; p < kFitRing; ++p) mma(p);
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < C; ++j) {
      if (ct0 + j >= CT) continue;
      f32x4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (BWD) {
          const float h = a.round_h ? (float)(T)e[i][j][r] : e[i][j][r];
          v[r] = acc[i][j][r] * (1.0f - h * h);
        } else {
          v[r] = act_tanh(acc[i][j][r] + e[i][0][r]);
        }
      }
      const int64_t ct = ct0 + j;
      if constexpr (BWD) {
        if (EVAL || l > 1) panel_store<P>(a, (T*)(par ? a.pp0 : a.pp1), ct, rt0 + i, lane, v);
        if constexpr (!EVAL)
          ((f32x4*)a.act)[fit_block(a, l - 1, ct, rt0 + i) + dw_slot(lane)] = quad_transpose(v, lane);
      } else {
        const int64_t o = fit_block(a, l, ct, rt0 + i);
        ((f32x4*)a.act)[o + lane] = v;
        if constexpr (!EVAL) ((f32x4*)a.hx)[o + dw_slot(lane)] = quad_transpose(v, lane);
        if (last) {
          f32x4 dl;
#pragma unroll
          for (int r = 0; r < 4; ++r) dl[r] = wo[i][r] * (1.0f - v[r] * v[r]);
          panel_store<P>(a, (T*)a.pp2, ct, rt0 + i, lane, dl);
        }
        if constexpr (sizeof(T) == 2) {
          if (l + 1 < a.mp.nh) panel_store<P>(a, (T*)((l & 1) ? a.pp1 : a.pp0), ct, rt0 + i, lane, v);
        }
      }
    }
}

// Closing kernel of a layer-by-layer evaluation: one column tile per workgroup takes the network's
// output from h_{nh-1}, d out / d t from delta_0 and assembles log pi and its gradient, in the
// tile engine's order throughout.  Bound by latency, like the layers of a small batch (64 points of
// 12 -> 512 x 4: 6.3 us here, 3.5 us a layer; one tile per CU through all weights took 41 us, the eight
// kernels take 28).
template <class P>
__global__ __launch_bounds__(kThreads) void eval_close_kernel(KArgs a, FitArgs f) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using T = typename P::T;
  const int64_t ct = blockIdx.x, c0 = ct * 16;
  const int mv = (int)((a.st.N - c0) < 16 ? (a.st.N - c0) : 16);
  const int nh = a.mp.nh;
  const T* d0 = (const T*)(((nh - 2) & 1) ? f.pp0 : f.pp1) + ct * 16 * a.mp.H;
  const PanelEval<T> pe{f.act + fit_block(f, nh - 1, ct, 0) * 4, d0,
                        a.tg.gprec, generic_ptr((double*)(smem + a.lds.cst))};
  a.tg.gprec = pe.gp;
  eval_tile<P, 1>(a, smem, nullptr, TView{const_cast<double*>(a.ex_x) + c0, a.ex_pitch}, mv,
                  a.ex_lp + c0, TView{a.ex_g ? a.ex_g + c0 : nullptr, a.ex_pitch},
                  a.ex_grad != 0, true, false, pe);
}

// Network output, upstream gradient (training: 2 (out - y) / n and the loss; target points: the
// weights) and delta_L = u w_out (1 - h_L^2) of one column tile per workgroup.  The output dot
// product runs in the tile engine's order: wave w sums the rows of its H / waves share, lane groups
// by butterfly, waves in order.
template <class P>
__global__ __launch_bounds__(kThreads) void fit_output_kernel(FitArgs a) {
  __shared__ float outp[kWaves][16], ups[16];
  __shared__ double r2[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, cl = lane & 15;
  const int H = a.mp.H, RTW = H / (16 * kWaves), L = a.mp.nh - 1;
  const int64_t ct = blockIdx.x;
  const float* __restrict__ Wo = (const float*)a.mp.wout;
  f32x4* hL = (f32x4*)a.act + fit_block(a, L, ct, 0);
  if (a.t_in) {
    float po = 0;
#pragma unroll 4
    for (int rr = 0; rr < RTW; ++rr) {
      const int rt = wv * RTW + rr;
      const f32x4 wo = *(const f32x4*)(Wo + rt * 16 + 4 * g), h = hL[rt * 64 + lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) po += wo[r] * h[r];
    }
    const float v = sum_lane_groups(po);
    if (g == 0) outp[wv][cl] = v;
    __syncthreads();
  }
  if (tid < 16) {
    const int64_t c = ct * 16 + tid;
    float u = 0.f;
    double r = 0;
    if (a.t_in) {
      float o = outp[0][tid];
      for (int w = 1; w < kWaves; ++w) o += outp[w][tid];
      o = o + Wo[H];
      if (c < a.n) r = (double)o - (double)a.y[a.perm[a.batch0 + c]];
      u = (float)(2.0 * r / (double)a.n_batch);
    } else if (c < a.n) {
      bool use = a.tg.plain_mode == 0;
      if (a.tg.plain_mode == 1) {
        use = true;
        for (int i = 0; i < a.mp.d; ++i) {
          const double xv = a.x[i * a.x_pitch + c];
          use = use && xv >= a.tg.train_lo[i] && xv <= a.tg.train_hi[i];
        }
      }
      u = use ? (float)(a.tg.mlp_coef * (a.upstream ? a.upstream[c] : 1.0)) : 0.f;
    }
    ups[tid] = u;
    a.up[c] = u;
    r2[tid] = r * r;
  }
  __syncthreads();
  if (a.t_in && tid == 0) {
    double s = 0;
    for (int c = 0; c < 16; ++c) s += r2[c];
    a.loss_part[ct] = s;
  }
  const float u = ups[cl];
  for (int rr = 0; rr < RTW; ++rr) {
    const int rt = wv * RTW + rr;
    const f32x4 wo = *(const f32x4*)(Wo + rt * 16 + 4 * g), h4 = hL[rt * 64 + lane];
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float h = a.round_h ? (float)(typename P::T)h4[r] : h4[r];
      v[r] = u * wo[r] * (1.0f - h * h);
    }
    if (L > 0) panel_store<P>(a, (typename P::T*)a.pp0, ct, rt, lane, v);
    hL[rt * 64 + dw_slot(lane)] = quad_transpose(v, lane);
  }
}

}  // namespace best
