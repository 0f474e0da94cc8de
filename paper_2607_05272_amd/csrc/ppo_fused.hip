// ppo_fused.hip -- the policy-gradient minibatch (paper Sec. 4.3) of the policy networks the
// rollouts use, in four launches (see ppo_kernels.hip for the definition of the loss, the
// roundings and the hi + lo gradient operands, and for networks of other widths):
//   gather   the samples' indices, observations and scalars; the weights into operand order
//   mlp      per workgroup of 16 RT samples: forward, loss and backward through every layer
//            with the activations in LDS and GELU'(z) in registers
//   wgrad    G_l = A_{l-1}^T dZ_l over chunks of the samples
//   finish   the chunks', the bias gradients' and the loss terms' sums in a fixed order, and in
//            an update Adam's step with the weights' rewrite (302 us per 8 minibatches of 4096 of
//            the 32-256-256-25 network with launches of their own, 269 us so)
// Nothing but the operands of the weight products passes between the launches through memory;
// with a launch per layer and elementwise step (ppo_kernels.hip) a minibatch of 8192 samples of
// the 64-256-256-49 network took 124 us, here 45; 16384 of the 96-512-512-97 one 475 and 156 us.
// Per sample both forms compute the same bits up to GELU'; the sums over samples differ in order.
#include "ppo_dev.hpp"
#include "train_dev.hpp"

namespace bsim {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4v;

// Operands of the MFMAs in fragment order: for a tile of 16 rows (units) and a step of KS
// contraction indices, the 64 lanes' KL elements lie back to back, lane = kq 16 + row holding
// indices kq KL .. + KL - 1 of the step, so a wave's fragment load is one contiguous block.
// Tiles are tile-major, then steps.
//
// Stores contraction indices k0 + dk .. + 3 (both multiples of 4, k0 of 16 with a tile and a k0
// that a wave's lanes share, dk < 16) of row r16 of a tile, of `steps` steps.
template <class Md>
__device__ __forceinline__ void frag_store4(typename Md::T* base, int steps, int tile, int r16,
                                            int k0, int dk, typename Md::four v) {
  if constexpr (Md::KL == 8) {
    typename Md::T* p = base + ((size_t)tile * steps + k0 / 32) * 512 + (k0 & 16) * 16;
    *reinterpret_cast<typename Md::four*>(p + (dk >> 3) * 128 + r16 * 8 + (dk & 4)) = v;
  } else {
    typename Md::T* p = base + ((size_t)tile * steps + k0 / 4) * 64;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[(dk >> 2) * 64 + i * 16 + r16] = v[i];
  }
}

// ---- gather -----------------------------------------------------------------------------------
struct SampleIn {
  float adv, ret, logp_old;
  int act;   // -1 for the padding past M
};

// One weight matrix into fragment order: element (k, n) of the operand is src[k sk + n sn] for
// k < kv and n < nv, zero in the padding to K x N.
template <class Md>
struct PackSeg {
  const typename Md::T* src;
  typename Md::T* dst;
  int K, N, sk, sn, kv, nv;
  int first;   // first fragment lane of this matrix
};
constexpr int kPackSegs = 5;
template <class Md>
struct GatherArgs {
  uint64_t seed;
  int M, Mp, T, E, F, F64, reinforce;
  const float* obs;
  const uint8_t* act;
  const float* logp_old;
  const double *adv, *ret;
  int64_t* idx_out;
  SampleIn* in;             // [Mp]
  typename Md::T *X, *Xf;   // [Mp][F64] and its fragments over the samples
  int npack;                // fragment lanes of all matrices
  PackSeg<Md> seg[kPackSegs];
};

// kGatherRows samples per workgroup, its observations' loads all in flight at once: they are
// single words of separate cache lines (E words apart), which bounds this kernel: 8192 x 64
// words in 15 us, 16384 x 96 in 35, about 40 lines a nanosecond. 256 threads with twice the loads
// each or 1024 with half take 3 us longer. The workgroups past the samples pack the weights.
constexpr int kGatherRows = 32, kGatherThr = 512, kMaxF64 = 128;
template <class Md>
__global__ __launch_bounds__(kGatherThr) void pg_gather_k(GatherArgs<Md> g) {
  typedef typename Md::T T;
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= g.Mp / kGatherRows) {   // uniform per workgroup
    const int q = (blockIdx.x - g.Mp / kGatherRows) * kGatherThr + tid;
    if (q >= g.npack) return;
    int sidx = 0;
#pragma unroll
    for (int i = 1; i < kPackSegs; ++i)
      if (q >= g.seg[i].first) sidx = i;
    const PackSeg<Md> s = g.seg[sidx];
    const int f = q - s.first, lane = f & 63, steps = s.K / Md::KS;
    const int step = (f >> 6) % steps, tile = (f >> 6) / steps;
    const int n = tile * 16 + (lane & 15), k0 = step * Md::KS + (lane >> 4) * Md::KL;
    T v[Md::KL];
#pragma unroll
    for (int j = 0; j < Md::KL; ++j)
      v[j] = k0 + j < s.kv && n < s.nv ? s.src[(size_t)(k0 + j) * s.sk + (size_t)n * s.sn] : T(0);
    T* d = s.dst + (size_t)f * Md::KL;
    if constexpr (Md::KL == 8) {
      u32x4v w;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = (uint32_t)v[2 * j] | ((uint32_t)v[2 * j + 1] << 16);
      *reinterpret_cast<u32x4v*>(d) = w;
    } else {
      d[0] = v[0];
    }
    return;
  }
  __shared__ int ts[kGatherRows], es[kGatherRows];
  __shared__ float xs[kGatherRows][kMaxF64 + 1];
  const int m0 = blockIdx.x * kGatherRows;
  size_t ti = 0;
  bool live = false;
  if (tid < kGatherRows) {
    const int m = m0 + tid;
    int tt = -1, ee = 0;
    live = m < g.M;
    if (live) {
      const u32x4 w = draw(g.seed, (uint32_t)m, 0xFFFFFFFDu, P_MINIBATCH, 0, 0);
      const double n = (double)g.T * (double)g.E;
      long long i = (long long)(unit(w.x, w.y) * n);
      if (i > (long long)g.T * g.E - 1) i = (long long)g.T * g.E - 1;
      if (g.idx_out) g.idx_out[m] = i;
      ti = (size_t)i;
      tt = (int)i / g.E;   // T E < 2^31 (checked by the host)
      ee = (int)i - tt * g.E;
    }
    ts[tid] = tt;
    es[tid] = ee;
  }
  __syncthreads();
  constexpr int kIt = kGatherRows * kMaxF64 / kGatherThr;
  float v[kIt];
  const int n = kGatherRows * g.F64;
#pragma unroll
  for (int j = 0; j < kIt; ++j) {
    const int q = tid + j * kGatherThr;
    v[j] = 0.f;
    if (q < n) {
      const int sl = q / g.F64, f = q % g.F64;
      if (ts[sl] >= 0 && f < g.F) v[j] = g.obs[((size_t)ts[sl] * g.F + f) * g.E + es[sl]];
    }
  }
  if (tid < kGatherRows) {
    SampleIn s{0.f, 0.f, 0.f, -1};
    if (live) {
      s.act = g.act[ti];
      s.adv = (float)g.adv[ti];
      s.ret = (float)g.ret[ti];
      if (!g.reinforce) s.logp_old = g.logp_old[ti];
    }
    g.in[m0 + tid] = s;
  }
#pragma unroll
  for (int j = 0; j < kIt; ++j) {
    const int q = tid + j * kGatherThr;
    if (q < n) {
      const int sl = q / g.F64, f = q % g.F64;
      const float x = Md::actf(v[j]);
      g.X[(size_t)(m0 + sl) * g.F64 + f] = Md::act(x);
      xs[sl][f] = x;
    }
  }
  __syncthreads();
  const int steps = g.Mp / Md::KS;
  for (int q = tid; q < g.F64 * (kGatherRows / 4); q += kGatherThr) {
    const int f = q % g.F64, s4 = 4 * (q / g.F64);
    const float w[4] = {xs[s4][f], xs[s4 + 1][f], xs[s4 + 2][f], xs[s4 + 3][f]};
    frag_store4<Md>(g.Xf, steps, f >> 4, f & 15, m0 + (s4 & ~15), s4 & 15, Md::pack(w));
  }
}

// ---- forward, loss and backward of 16 RT samples -------------------------------------------------
// Bound by vector issue (GELU, its derivative, the packing of what the weight products read:
// half of the cycles at 8192 samples of the 64-256-256-49 network, 16.5 us) and by the chain of
// barrier-separated layers (the matrix cores are busy for a seventh of it). Each wave keeps
// GELU'(z) of its units in registers from the forward to the backward pass, so a workgroup
// holds as many samples as the registers of its widest layer allow: 16 waves of 128 registers
// for the 256-wide networks (42.0 us per minibatch with 8 waves, 41.0 with 16), 8 of 256 for 32
// samples of the 512-wide one (167 against 200 with 16, which spill).
//
// The weight fragments of TPW output tiles (tile0 + i tstride) over K, read from L2 in fragment
// order D steps ahead of their use; start() issues the first D (before the barrier that the
// activations wait for, so that their latency passes under the previous phase).
template <class Md, int K, int TPW>
struct Weights {
  static constexpr int KSN = K / Md::KS, DEPTH = 4, D = KSN < DEPTH ? KSN : DEPTH,
                       S = D + 1;
  typename Md::frag w[S][TPW];
  const typename Md::T* wp[TPW];
  __device__ __forceinline__ void load(int ks) {
#pragma unroll
    for (int i = 0; i < TPW; ++i) w[ks % S][i] = Md::load(wp[i] + (size_t)ks * 64 * Md::KL);
  }
  __device__ __forceinline__ void start(const typename Md::T* W, int tile0, int tstride) {
#pragma unroll
    for (int i = 0; i < TPW; ++i)
      wp[i] = W + ((size_t)(tile0 + i * tstride) * KSN * 64 + (threadIdx.x & 63)) * Md::KL;
#pragma unroll
    for (int ks = 0; ks < D; ++ks) load(ks);
  }
};

// acc[i][rt] = act[rows rt0 + rt] W[:, tile i] over K: activations (one or two terms) from LDS
// rows of stride sa, one step ahead; the scheduling barriers keep the loads from sinking to
// their uses.
template <class Md, int K, int TPW, int RTN, int SPL>
__device__ __forceinline__ void mlp_mma(const typename Md::T* hi, const typename Md::T* lo, int sa,
                                        Weights<Md, K, TPW>& W, int rt0, f32x4 (&acc)[TPW][RTN]) {
  typedef typename Md::frag Fr;
  typedef Weights<Md, K, TPW> Wt;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int rt = 0; rt < RTN; ++rt) acc[i][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int ao = (rt0 * 16 + (lane & 15)) * sa + Md::koff(lane);
  Fr b[2][SPL][RTN];
  auto load_act = [&](int slot, int ks) {
#pragma unroll
    for (int rt = 0; rt < RTN; ++rt) {
      b[slot][0][rt] = Md::load(hi + ao + rt * 16 * sa + ks * Md::KS);
      if constexpr (SPL == 2) b[slot][1][rt] = Md::load(lo + ao + rt * 16 * sa + ks * Md::KS);
    }
  };
  load_act(0, 0);
#pragma unroll
  for (int ks = 0; ks < Wt::KSN; ++ks) {
    if (ks + 1 < Wt::KSN) load_act((ks + 1) & 1, ks + 1);
    if (ks + Wt::D < Wt::KSN) W.load(ks + Wt::D);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < SPL; ++s)
#pragma unroll
      for (int rt = 0; rt < RTN; ++rt)
#pragma unroll
        for (int i = 0; i < TPW; ++i)
          acc[i][rt] = Md::mfma(b[ks & 1][s][rt], W.w[ks % Wt::S][i], acc[i][rt]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// sum and maximum over the 16 lanes of a DPP row, in every lane of it (rotations by 8, 4, 2, 1:
// both operands of each step are the same pair in the lanes that share it, so all lanes agree)
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f<0x128>(v);
  v += dpp_f<0x124>(v);
  v += dpp_f<0x122>(v);
  return v + dpp_f<0x121>(v);
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_f<0x128>(v));
  v = fmaxf(v, dpp_f<0x124>(v));
  v = fmaxf(v, dpp_f<0x122>(v));
  return fmaxf(v, dpp_f<0x121>(v));
}

// The sum over a sample's outputs, output p + 16 i in lane p: outputs 64 apart, then 32, 16 and
// the rest, the order of a butterfly over 64 lanes holding outputs i and i + 64 (mb_loss_k's), so
// that the log-probabilities of both forms are the same bits.
template <int N>
__device__ __forceinline__ float out_sum(const float (&v)[N]) {
  static_assert(N == 4 || N == 8, "64 or 128 outputs");
  float x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = N == 8 ? v[i] + v[(i + 4) % N] : v[i];
  return row16_sum((x[0] + x[2]) + (x[1] + x[3]));
}

template <class Md>
struct MlpArgs {
  typedef typename Md::T T;
  int M, Mp, A, Ap, reinforce;
  float clip, c_v, c_h;
  const SampleIn* in;
  const T* X;
  const T *W1f, *W2f, *W3f, *W3b, *W2b;   // fragment order (forward W1, W2, W3; backward W3, W2)
  const float *b1, *b2, *b3;
  T *H1f, *H2f;                            // activations' fragments over the samples
  T *dO[2], *dZ2[2], *dZ1[2];              // gradients' fragments over the samples, hi and lo
  float* col;                              // [workgroups][AK + H2 + H1] bias gradients' sums
  double* terms;                           // [workgroups][3] policy, value, entropy sums
  uint32_t* err;
};

template <class Md, int FK, int H1, int H2, int AK, int RT>
struct MlpLds {
  static constexpr int ROWS = 16 * RT, HM = H1 > H2 ? H1 : H2;
  static constexpr int SX = FK + Md::PAD, SH = HM + Md::PAD, SO = AK + Md::PAD, SL = AK + 4;
  static constexpr size_t e = sizeof(typename Md::T);
  static constexpr size_t max(size_t a, size_t b) { return a > b ? a : b; }
  static constexpr size_t X = max(ROWS * SX * e, ROWS * SO * e * Md::SPLIT);   // x, then dO
  static constexpr size_t Q = max(ROWS * SH * e, ROWS * SL * 4);   // h1, then out, then dZ2 hi
  static constexpr size_t R = ROWS * SH * e;                       // h2, then dZ2 lo
  static constexpr size_t T = ROWS * 3 * 8;                        // loss terms per sample
  static constexpr size_t LDS = X + Q + R + T;
};

template <class Md, int FK, int H1, int H2, int AK, int RT, int NW>
__global__ __launch_bounds__(NW * 64) void pg_mlp_k(MlpArgs<Md> a) {
  typedef typename Md::T T;
  typedef MlpLds<Md, FK, H1, H2, AK, RT> L;
  constexpr int ROWS = L::ROWS, NTHR = NW * 64;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* xs = reinterpret_cast<T*>(smem);
  T* do_hi = xs;
  T* do_lo = xs + ROWS * L::SO;
  T* h1s = reinterpret_cast<T*>(smem + L::X);
  float* outs = reinterpret_cast<float*>(smem + L::X);
  T* dz_hi = h1s;
  T* h2s = reinterpret_cast<T*>(smem + L::X + L::Q);
  T* dz_lo = h2s;
  double* tsum = reinterpret_cast<double*>(smem + L::X + L::Q + L::R);
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, kq = lane >> 4;
  // in a scalar register, and with it the bases of the wave's weights and fragments
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * ROWS, steps = a.Mp / Md::KS;

  constexpr int T1 = H1 / 16 / NW, T2 = H2 / 16 / NW;
  static_assert(H1 % (16 * NW) == 0 && H2 % (16 * NW) == 0, "whole tiles per wave");
  // the output layer's AK / 16 tiles x RT row tiles over the waves, RTN row tiles each
  constexpr int NT = AK / 16, RTN = NT * RT > NW ? NT * RT / NW : 1;
  static_assert(RT % RTN == 0, "row-tile runs of the output layer");
  const bool out_wave = wave < NT * RT / RTN;
  const int otile = wave % NT, ort0 = (wave / NT) * RTN;

  // a wave's tiles of a layer in passes of P: tile wave + NW c for c = P g .. P g + P - 1
  constexpr int P1 = T1 < 2 ? 1 : 2, P2 = T2 < 2 ? 1 : 2;
  Weights<Md, FK, P1> w1;
  w1.start(a.W1f, wave, NW);
  // the scalars of the sample whose loss this thread's 16 lanes will take
  static_assert(ROWS <= NTHR / 16, "one pass over the samples in the loss");
  const int lrow = tid >> 4;
  SampleIn sin{0.f, 0.f, 0.f, -1};
  if (lrow < ROWS) sin = a.in[m0 + lrow];
  // the samples' observations, 16 bytes per load
  constexpr int V = 16 / sizeof(T);
  for (int q = tid; q < ROWS * FK / V; q += NTHR) {
    const int r = q / (FK / V), c = (q % (FK / V)) * V;
    *reinterpret_cast<u32x4v*>(xs + r * L::SX + c) =
        *reinterpret_cast<const u32x4v*>(a.X + (size_t)(m0 + r) * FK + c);
  }
  __syncthreads();

  // hidden layer: h = GELU(act W + b) into LDS (sample rows) and fragment order, GELU'(z) kept
  f32x4 gp1[T1][RT], gp2[T2][RT];
  auto hidden = [&](int c0, auto& acc, auto& gp, const float* bias, T* out, T* frag) {
    constexpr int N = sizeof(acc) / sizeof(acc[0]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int u = (wave + NW * (c0 + i)) * 16 + r16;
      const float b = bias[u];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int row = rt * 16 + kq * 4;
        // samples past M (M is a multiple of 4, and so is the lane's first row) are zero
        typename Md::four p = Md::hidden(acc[i][rt] + f32x4{b, b, b, b}, gp[c0 + i][rt]);
        if (m0 + row >= a.M) p = typename Md::four{};
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(row + q) * L::SH + u] = Md::get(p, q);
        frag_store4<Md>(frag, steps, wave + NW * (c0 + i), r16, m0 + rt * 16, kq * 4, p);
      }
    }
  };
  Weights<Md, H1, P2> w2;
#pragma unroll
  for (int c = 0; c < T1; c += P1) {
    f32x4 acc[P1][RT];
    mlp_mma<Md, FK, P1, RT, 1>(xs, nullptr, L::SX, w1, 0, acc);
    if (c + P1 < T1) w1.start(a.W1f, wave + NW * (c + P1), NW);
    else w2.start(a.W2f, wave, NW);
    hidden(c, acc, gp1, a.b1, h1s, a.H1f);
  }
  __syncthreads();
  Weights<Md, H2, 1> w3;
#pragma unroll
  for (int c = 0; c < T2; c += P2) {
    f32x4 acc[P2][RT];
    mlp_mma<Md, H1, P2, RT, 1>(h1s, nullptr, L::SH, w2, 0, acc);
    if (c + P2 < T2) w2.start(a.W2f, wave + NW * (c + P2), NW);
    else if (out_wave) w3.start(a.W3f, otile, 0);
    hidden(c, acc, gp2, a.b2, h2s, a.H2f);
  }
  __syncthreads();
  Weights<Md, AK, P2> w3b;
  if (out_wave) {
    f32x4 acc[1][RTN];
    mlp_mma<Md, H2, 1, RTN, 1>(h2s, nullptr, L::SH, w3, ort0, acc);
    const int u = otile * 16 + r16;
    const float b = u < a.Ap ? a.b3[u] : 0.f;
#pragma unroll
    for (int rt = 0; rt < RTN; ++rt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        outs[((ort0 + rt) * 16 + kq * 4 + q) * L::SL + u] = acc[0][rt][q] + b;
  }
  w3b.start(a.W3b, wave, NW);
  __syncthreads();
  // loss and dL/dout: 16 lanes per sample, lane p of them holding outputs p, p + 16, ...
  {
    constexpr int NA = AK / 16;
    if (const int r = lrow; r < ROWS) {   // whole rows of 16 lanes
      const int p = lane & 15;
      const SampleIn& s = sin;
      const float* l = outs + r * L::SL;
      const bool bad = s.act >= a.A;   // invalid stored action: flagged, contributes nothing
      if (bad && p == 0) atomicOr(a.err, ERR_ACTION);
      const bool on = s.act >= 0 && !bad;
      float v[NA], e[NA];
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        v[i] = l[p + 16 * i];
        if (p + 16 * i < a.A) mx = fmaxf(mx, v[i]);
      }
      mx = row16_max(mx);
#pragma unroll
      for (int i = 0; i < NA; ++i) e[i] = p + 16 * i < a.A ? expf(v[i] - mx) : 0.f;
      const float lS = logf(out_sum(e));
      float ph[NA];
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const float lp = (v[i] - mx) - lS;
        const bool in = p + 16 * i < a.A;
        e[i] = in ? expf(lp) : 0.f;
        ph[i] = in ? e[i] * lp : 0.f;
        v[i] = lp;
      }
      const float H = -out_sum(ph);
      const float logp = (l[on ? s.act : 0] - mx) - lS, val = l[a.A];
      const float invM = 1.0f / (float)a.M;
      float dlogp, pterm;
      policy_term(a.reinforce, a.clip, logp, s.logp_old, s.adv, invM, dlogp, pterm);
      const float dv = 2.0f * a.c_v * (val - s.ret) * invM;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int o = p + 16 * i;
        float g = 0.f;
        if (o < a.A) g = -dlogp * e[i] + a.c_h * invM * e[i] * (v[i] + H) + (o == s.act ? dlogp : 0.f);
        else if (o == a.A) g = dv;
        if (!on) g = 0.f;
        T hi, lo;
        Md::split(g, hi, lo);
        do_hi[r * L::SO + o] = hi;
        if (Md::SPLIT == 2) do_lo[r * L::SO + o] = lo;
      }
      if (p == 0) {
        tsum[r * 3] = on ? (double)pterm : 0.0;
        tsum[r * 3 + 1] = on ? (double)(val - s.ret) * (double)(val - s.ret) : 0.0;
        tsum[r * 3 + 2] = on ? (double)H : 0.0;
      }
    }
  }
  __syncthreads();
  float* col = a.col + (size_t)blockIdx.x * (AK + H2 + H1);
  // hidden layer backward: dz = (dZ_next W^T) GELU'(z), its column sums, its fragments over the
  // samples and (kRows) its two terms as sample rows in LDS
  auto back = [&](int c0, auto& acc, auto& gp, T* hi_s, T* lo_s, T* const* frag, float* csum) {
    constexpr int N = sizeof(acc) / sizeof(acc[0]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int u = (wave + NW * (c0 + i)) * 16 + r16;
      float cs = 0.f;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int row = rt * 16 + kq * 4;
        float v[4], l[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q] = m0 + row < a.M ? acc[i][rt][q] * gp[c0 + i][rt][q] : 0.f;
          cs += v[q];
        }
        const typename Md::four hi = Md::pack(v);
#pragma unroll
        for (int q = 0; q < 4; ++q) l[q] = v[q] - Md::value(Md::get(hi, q));
        const typename Md::four lo = Md::pack(l);
        if (hi_s) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            hi_s[(row + q) * L::SH + u] = Md::get(hi, q);
            if (Md::SPLIT == 2) lo_s[(row + q) * L::SH + u] = Md::get(lo, q);
          }
        }
        frag_store4<Md>(frag[0], steps, wave + NW * (c0 + i), r16, m0 + rt * 16, kq * 4, hi);
        if (Md::SPLIT == 2) frag_store4<Md>(frag[1], steps, wave + NW * (c0 + i), r16, m0 + rt * 16, kq * 4, lo);
      }
      cs += __shfl_xor(cs, 16, 64);
      cs += __shfl_xor(cs, 32, 64);
      if (kq == 0) csum[u] = cs;
    }
  };
  Weights<Md, H2, P1> w2b;
#pragma unroll
  for (int c = 0; c < T2; c += P2) {
    f32x4 acc[P2][RT];
    mlp_mma<Md, AK, P2, RT, Md::SPLIT>(do_hi, do_lo, L::SO, w3b, 0, acc);
    if (c + P2 < T2) w3b.start(a.W3b, wave + NW * (c + P2), NW);
    else w2b.start(a.W2b, wave, NW);
    back(c, acc, gp2, dz_hi, dz_lo, a.dZ2, col + AK);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < T1; c += P1) {
    f32x4 acc[P1][RT];
    mlp_mma<Md, H2, P1, RT, Md::SPLIT>(dz_hi, dz_lo, L::SH, w2b, 0, acc);
    if (c + P1 < T1) w2b.start(a.W2b, wave + NW * (c + P1), NW);
    back(c, acc, gp1, nullptr, nullptr, a.dZ1, col + AK + H2);
  }
  // the loss terms' and b3's sums over the rows, and dO in fragment order
  if (tid < 3) {
    double s = 0.0;
    for (int r = 0; r < ROWS; ++r) s += tsum[r * 3 + tid];
    a.terms[(size_t)blockIdx.x * 3 + tid] = s;
  }
  for (int q = tid; q < AK * (ROWS / 4); q += NTHR) {
    const int o = q % AK, r = 4 * (q / AK);
#pragma unroll
    for (int s = 0; s < Md::SPLIT; ++s) {
      const T* d = s == 0 ? do_hi : do_lo;
      float w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = Md::value(d[(r + i) * L::SO + o]);
      frag_store4<Md>(a.dO[s], steps, o >> 4, o & 15, m0 + (r & ~15), r & 15, Md::pack(w));
    }
  }
  if (tid < AK) {
    float s = 0.f;
#pragma unroll 8
    for (int r = 0; r < ROWS; ++r) {
      s += Md::value(do_hi[r * L::SO + tid]);
      if (Md::SPLIT == 2) s += Md::value(do_lo[r * L::SO + tid]);
    }
    col[tid] = s;
  }
}

// ---- weight gradients --------------------------------------------------------------------------
// A 64 x 64 tile of one layer's gradient over a chunk of the samples per workgroup: every wave
// takes every fourth step of the chunk with 4 x 4 MFMA tiles of its own (12 fragments feed 32
// MFMAs: a third of the operand traffic of one 32 x 32 tile per wave), and the four waves'
// tiles are added in a fixed order through LDS. Bound by the operands' way from L2: 9 us for
// 8192 samples of the 64-256-256-49 network, 39 us for 16384 of the 96-512-512-97 one (21 and 150
// with 32 x 32 tiles and unit-major operands).
template <class Md>
struct WgLayer {
  const typename Md::T *A, *B0, *B1;   // fragments over the samples: input units; output units
  float* P;                            // [S][R64][N64] partial products
  int R64, N64, first;                 // first workgroup of this layer
};
template <class Md>
struct WgArgs {
  WgLayer<Md> l[3];
  int steps, chunk, S;                 // steps of the samples, per chunk (a multiple of 4), chunks
};
constexpr int kWgStride = 68;          // LDS row stride: 4-row groups of a store on separate banks
template <class Md>
__global__ __launch_bounds__(256) void pg_wgrad_k(WgArgs<Md> g) {
  typedef typename Md::frag Fr;
  __shared__ __attribute__((aligned(16))) float part[2][64 * kWgStride];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const WgLayer<Md> L = g.l[b >= g.l[2].first ? 2 : b >= g.l[1].first ? 1 : 0];
  const int q = b - L.first, z = q % g.S, tile = q / g.S, tn = L.N64 / 64;
  const int ty = tile / tn, tx = tile % tn;
  const size_t row = (size_t)g.steps * 64 * Md::KL;   // one 16-unit tile's fragments
  const typename Md::T* A = L.A + (size_t)ty * 4 * row + (size_t)lane * Md::KL;
  const typename Md::T* B0 = L.B0 + (size_t)tx * 4 * row + (size_t)lane * Md::KL;
  const typename Md::T* B1 = L.B1 + (size_t)tx * 4 * row + (size_t)lane * Md::KL;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int k1 = min(z * g.chunk + g.chunk, g.steps);
  Fr fa[4], fb[4], fl[4], na[4], nb[4], nl[4];
  auto load = [&](int k, Fr (&x)[4], Fr (&y)[4], Fr (&w)[4]) {
    const size_t o = (size_t)k * 64 * Md::KL;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = Md::load(A + i * row + o);
      y[i] = Md::load(B0 + i * row + o);
      if constexpr (Md::SPLIT == 2) w[i] = Md::load(B1 + i * row + o);
    }
  };
  int k = z * g.chunk + wave;
  if (k < k1) load(k, na, nb, nl);
  for (; k < k1; k += 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { fa[i] = na[i]; fb[i] = nb[i]; fl[i] = nl[i]; }
    if (k + 4 < k1) load(k + 4, na, nb, nl);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = Md::mfma(fa[i], fb[j], acc[i][j]);
    if constexpr (Md::SPLIT == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = Md::mfma(fa[i], fl[j], acc[i][j]);
    }
  }
  // waves 2 and 3 into LDS, added by waves 0 and 1; the two sums into LDS, added on the way out
  auto at = [&](int i, int j, int r) {
    return (16 * i + 4 * (lane >> 4) + r) * kWgStride + 16 * j + (lane & 15);
  };
  auto put = [&](float* d) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) d[at(i, j, r)] = acc[i][j][r];
  };
  if (wave >= 2) put(part[wave - 2]);
  __syncthreads();
  if (wave < 2) {
    float* d = part[wave];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) d[at(i, j, r)] += acc[i][j][r];
  }
  __syncthreads();
  float* P = L.P + (size_t)z * L.R64 * L.N64 + (size_t)ty * 64 * L.N64 + tx * 64;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 16 * i + (threadIdx.x >> 4), c = 4 * (threadIdx.x & 15);
    *reinterpret_cast<f32x4*>(P + (size_t)r * L.N64 + c) =
        *reinterpret_cast<const f32x4*>(&part[0][r * kWgStride + c]) +
        *reinterpret_cast<const f32x4*>(&part[1][r * kWgStride + c]);
  }
}

// ---- the gradients' and the loss's final sums ------------------------------------------------------
struct FinLayer {
  const float* P;
  int R64, N64, R, N;
  int first, goff;      // first entry in the flattened range; offset in the gradient vector
};
struct FinArgs {
  FinLayer l[3];
  int S, nent, nred;    // chunks, weight entries, workgroups that sum them
  const float* col;     // [nwg][width] bias partial sums: AK outputs, H2, H1 units
  int nwg, width, AK, H2, Ap;
  int boff[3];          // offsets of b3, b2, b1 in the gradient vector
  const double* terms;  // [nwg][3]
  int M;
  float c_v, c_h;
  double* loss;         // total, policy, value, entropy
  float* grads;
  AdamStep adam;        // p NULL: the gradient is written
};
constexpr int kFinThr = 256, kColUnits = 16, kColParts = kFinThr / kColUnits;
__global__ __launch_bounds__(kFinThr) void pg_finish_k(FinArgs a) {
  const int tid = threadIdx.x, b = blockIdx.x;
  if (b < a.nred) {   // weight entries: chunks in order
    const int q = b * kFinThr + tid;
    if (q >= a.nent) return;
    const FinLayer d = a.l[q >= a.l[2].first ? 2 : q >= a.l[1].first ? 1 : 0];
    const int e = q - d.first, r = e / d.N, c = e % d.N;
    const float* p = d.P + (size_t)r * d.N64 + c;
    const size_t st = (size_t)d.R64 * d.N64;
    float s = 0.f;
#pragma unroll 8
    for (int z = 0; z < a.S; ++z) s += p[z * st];
    finish_param(a.adam, a.grads, (size_t)(d.goff + e), s);
    return;
  }
  if (b < (int)gridDim.x - 1) {
    // bias gradients: kColUnits units per workgroup, part t of them adding workgroups t,
    // t + kColParts, ... in order, then the parts in order
    __shared__ float part[kColParts][kColUnits + 1];
    const int u = (b - a.nred) * kColUnits + tid % kColUnits, t = tid / kColUnits;
    float s = 0.f;
    if (u < a.width) {
#pragma unroll 8
      for (int w = t; w < a.nwg; w += kColParts) s += a.col[(size_t)w * a.width + u];
    }
    part[t][tid % kColUnits] = s;
    __syncthreads();
    if (t == 0 && u < a.width) {
#pragma unroll
      for (int i = 1; i < kColParts; ++i) s += part[i][tid];
      const int k = u < a.AK ? 0 : u < a.AK + a.H2 ? 1 : 2;
      const int i = k == 0 ? u : k == 1 ? u - a.AK : u - a.AK - a.H2;
      if (k > 0 || i < a.Ap) finish_param(a.adam, a.grads, (size_t)(a.boff[k] + i), s);
    }
    return;
  }
  // the last workgroup: loss terms, thread t adding workgroups t, t + kFinThr, ... in order,
  // then a pairwise tree
  __shared__ double dp[3][kFinThr];
  double s[3] = {0.0, 0.0, 0.0};
  for (int w = tid; w < a.nwg; w += kFinThr)
    for (int c = 0; c < 3; ++c) s[c] += a.terms[(size_t)w * 3 + c];
  for (int c = 0; c < 3; ++c) dp[c][tid] = s[c];
  __syncthreads();
  for (int w = kFinThr / 2; w > 0; w >>= 1) {
    if (tid < w)
      for (int c = 0; c < 3; ++c) dp[c][tid] += dp[c][tid + w];
    __syncthreads();
  }
  if (tid == 0) {
    const double pi = dp[0][0] / a.M, v = a.c_v * dp[1][0] / a.M, h = -a.c_h * dp[2][0] / a.M;
    a.loss[0] = pi + v + h;
    a.loss[1] = pi;
    a.loss[2] = v;
    a.loss[3] = h;
  }
}

// ---- host ------------------------------------------------------------------------------------------
int pad64(int x) { return (x + 63) & ~63; }

// Up to this many samples a workgroup of the mlp launch takes 16 of them, else 32: below, the
// launch lasts as long as one workgroup's chain of layers and the chip has room for more of
// them (4096 samples of the 64-256-256-49 network: 30 against 33 us per minibatch, 2048 of the
// 96-512-512-97 one 44 against 57); above, the weights are read from L2 half as often (8192:
// 42 against 46 us; 16384 of the wide network 150 against 172). fp32 networks are small and always
// take 16.
constexpr int kRtSmallM = 4096;
// Workgroups of the weight-gradient launch (16384 samples of the wide network, per minibatch:
// 256 158 us, 384 149, 512 154, 1024 160; 8192 of the 256-wide one: 42.3, 42.3, 49, 46). More
// than four chunks are rounded up to a multiple of eight, so that a chunk's workgroups land
// on one XCD and share its operands in that L2 (5 chunks 167 us, 8 chunks 154).
constexpr int kWgTarget = 384;

struct Plan {
  int Mp, F64, H1, H2, AK, rows, nwg, steps, chunk, S;
  size_t bytes;
  // offsets in the scratch
  size_t in, X, Xf, W1f, W2f, W3f, W3b, W2b, H1f, H2f, dO[2], dZ2[2], dZ1[2], col, terms, P[3];
};

Plan plan_of(const MlpParams& m, int M) {
  Plan p;
  const int ks = m.bf16 ? 32 : 4, two = m.bf16 ? 2 : 1;
  const size_t e = m.bf16 ? 2 : 4;
  p.Mp = pad64(M); p.F64 = pad64(m.F); p.H1 = m.H1; p.H2 = m.H2; p.AK = pad64(m.Ap);
  p.rows = !m.bf16 || M <= kRtSmallM ? 16 : 32;
  p.nwg = p.Mp / p.rows;
  p.steps = p.Mp / ks;
  const int tiles = (p.H2 * p.AK + p.H1 * p.H2 + p.F64 * p.H1) / 4096;
  int s = kWgTarget / tiles;
  if (s < 1) s = 1;
  if (s > 4) s = (s + 7) & ~7;
  p.chunk = ((p.steps + s - 1) / s + 3) & ~3;
  p.S = (p.steps + p.chunk - 1) / p.chunk;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) & ~(size_t)255;
    return o;
  };
  const size_t Mp = p.Mp;
  p.in = take(Mp * sizeof(SampleIn));
  p.X = take(Mp * p.F64 * e);
  p.Xf = take(Mp * p.F64 * e);
  p.W1f = take((size_t)p.F64 * p.H1 * e);
  p.W2f = take((size_t)p.H1 * p.H2 * e);
  p.W3f = take((size_t)p.H2 * p.AK * e);
  p.W3b = take((size_t)p.AK * p.H2 * e);
  p.W2b = take((size_t)p.H2 * p.H1 * e);
  p.H1f = take(Mp * p.H1 * e);
  p.H2f = take(Mp * p.H2 * e);
  for (int i = 0; i < two; ++i) {
    p.dO[i] = take(Mp * p.AK * e);
    p.dZ2[i] = take(Mp * p.H2 * e);
    p.dZ1[i] = take(Mp * p.H1 * e);
  }
  if (two == 1) p.dO[1] = p.dZ2[1] = p.dZ1[1] = 0;
  p.col = take((size_t)p.nwg * (p.AK + p.H2 + p.H1) * 4);
  p.terms = take((size_t)p.nwg * 3 * 8);
  p.P[0] = take((size_t)p.S * p.H2 * p.AK * 4);
  p.P[1] = take((size_t)p.S * p.H1 * p.H2 * 4);
  p.P[2] = take((size_t)p.S * p.F64 * p.H1 * 4);
  p.bytes = off;
  return p;
}

template <class Md, int FK, int H1, int H2, int AK, int RT, int NW>
hipError_t launch_mlp(const MlpArgs<Md>& a, int nwg, hipStream_t st) {
  typedef MlpLds<Md, FK, H1, H2, AK, RT> L;
  static_assert(L::LDS <= 160 * 1024, "LDS budget");
  auto kern = pg_mlp_k<Md, FK, H1, H2, AK, RT, NW>;
  static std::atomic<uint64_t> lds_on{0};
  const hipError_t e = allow_lds((const void*)kern, L::LDS, lds_on);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(nwg), dim3(NW * 64), L::LDS, st, a);
  return hipGetLastError();
}

// the networks of the rollout policies, padded: f(shape) or hipErrorNotSupported
template <class Md, int F, int A, int B, int O, int W1, int W2>
struct Net {
  typedef Md Mode;
  static constexpr int FK = F, H1 = A, H2 = B, AK = O, NW1 = W1, NW2 = W2;
};
template <class Fn>
hipError_t with_net(const MlpParams& m, Fn&& f) {
  const int F = pad64(m.F), O = pad64(m.Ap);
  auto is = [&](int bf, int a, int b, int c, int d) {
    return m.bf16 == bf && F == a && m.H1 == b && m.H2 == c && O == d;
  };
  if (is(0, 64, 64, 64, 64)) return f(Net<F32Mode, 64, 64, 64, 64, 4, 4>{});
  if (is(1, 64, 128, 128, 64)) return f(Net<Bf16Mode, 64, 128, 128, 64, 8, 8>{});
  if (is(1, 64, 256, 256, 64)) return f(Net<Bf16Mode, 64, 256, 256, 64, 16, 16>{});
  if (is(1, 128, 512, 512, 128)) return f(Net<Bf16Mode, 128, 512, 512, 128, 16, 8>{});
  return hipErrorNotSupported;
}

template <class N>
hipError_t run(const MlpParams& m, const void* d_weights, const size_t off[6], int T,
               const float* obs, const uint8_t* act, const float* logp_old, const double* adv,
               const double* ret, int M, uint64_t seed, float clip, float c_v, float c_h,
               int reinforce, void* scratch, double* loss_out, float* grads, const AdamStep* adam,
               int64_t* idx_out, uint32_t* err, hipStream_t st) {
  typedef typename N::Mode Md;
  typedef typename Md::T TT;
  const Plan p = plan_of(m, M);
  unsigned char* sb = static_cast<unsigned char*>(scratch);
  const unsigned char* wb = static_cast<const unsigned char*>(d_weights);
  auto at = [&](size_t o) { return reinterpret_cast<TT*>(sb + o); };
  const TT* w1 = reinterpret_cast<const TT*>(wb + off[0]);
  const TT* w2 = reinterpret_cast<const TT*>(wb + off[2]);
  const TT* w3 = reinterpret_cast<const TT*>(wb + off[4]);
  GatherArgs<Md> g;
  g.seed = seed; g.M = M; g.Mp = p.Mp; g.T = T; g.E = m.E; g.F = m.F; g.F64 = p.F64;
  g.reinforce = reinforce;
  g.obs = obs; g.act = act; g.logp_old = logp_old; g.adv = adv; g.ret = ret; g.idx_out = idx_out;
  g.in = reinterpret_cast<SampleIn*>(sb + p.in);
  g.X = at(p.X); g.Xf = at(p.Xf);
  // forward operands W1 [F][H1], W2 [H1][H2], W3 [H2][Ap] as (k, n); backward W3^T, W2^T
  g.seg[0] = {w1, at(p.W1f), p.F64, p.H1, m.H1, 1, m.F, p.H1, 0};
  g.seg[1] = {w2, at(p.W2f), p.H1, p.H2, m.H2, 1, p.H1, p.H2, 0};
  g.seg[2] = {w3, at(p.W3f), p.H2, p.AK, m.Ap, 1, p.H2, m.Ap, 0};
  g.seg[3] = {w3, at(p.W3b), p.AK, p.H2, 1, m.Ap, m.Ap, p.H2, 0};
  g.seg[4] = {w2, at(p.W2b), p.H2, p.H1, 1, m.H2, p.H2, p.H1, 0};
  int npack = 0;
  for (auto& s : g.seg) {
    s.first = npack;
    npack += s.K * s.N / Md::KL;
  }
  g.npack = npack;
  hipLaunchKernelGGL(pg_gather_k<Md>,
                     dim3(p.Mp / kGatherRows + (npack + kGatherThr - 1) / kGatherThr),
                     dim3(kGatherThr), 0, st, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  MlpArgs<Md> a;
  a.M = M; a.Mp = p.Mp; a.A = m.A; a.Ap = m.Ap; a.reinforce = reinforce;
  a.clip = clip; a.c_v = c_v; a.c_h = c_h;
  a.in = g.in; a.X = g.X;
  a.W1f = at(p.W1f); a.W2f = at(p.W2f); a.W3f = at(p.W3f); a.W3b = at(p.W3b); a.W2b = at(p.W2b);
  a.b1 = reinterpret_cast<const float*>(wb + off[1]);
  a.b2 = reinterpret_cast<const float*>(wb + off[3]);
  a.b3 = reinterpret_cast<const float*>(wb + off[5]);
  a.H1f = at(p.H1f); a.H2f = at(p.H2f);
  for (int i = 0; i < 2; ++i) { a.dO[i] = at(p.dO[i]); a.dZ2[i] = at(p.dZ2[i]); a.dZ1[i] = at(p.dZ1[i]); }
  a.col = reinterpret_cast<float*>(sb + p.col);
  a.terms = reinterpret_cast<double*>(sb + p.terms);
  a.err = err;
  if constexpr (Md::SPLIT == 2)
    e = p.rows == 16 ? launch_mlp<Md, N::FK, N::H1, N::H2, N::AK, 1, N::NW1>(a, p.nwg, st)
                     : launch_mlp<Md, N::FK, N::H1, N::H2, N::AK, 2, N::NW2>(a, p.nwg, st);
  else
    e = launch_mlp<Md, N::FK, N::H1, N::H2, N::AK, 1, N::NW1>(a, p.nwg, st);
  if (e != hipSuccess) return e;
  WgArgs<Md> w;
  FinArgs f;
  const TT* A_[3] = {a.H2f, a.H1f, g.Xf};
  TT* const* B_[3] = {a.dO, a.dZ2, a.dZ1};
  const int R64[3] = {p.H2, p.H1, p.F64}, N64[3] = {p.AK, p.H2, p.H1};
  const int R[3] = {p.H2, p.H1, m.F}, Nn[3] = {m.Ap, p.H2, p.H1};
  // gradient layout W1 [F][H1], b1, W2 [H1][H2], b2, W3 [H2][A'], b3
  const int gw1 = 0, gb1 = m.F * m.H1, gw2 = gb1 + m.H1, gb2 = gw2 + m.H1 * m.H2,
            gw3 = gb2 + m.H2, gb3 = gw3 + m.H2 * m.Ap;
  const int goff[3] = {gw3, gw2, gw1};
  int nblk = 0, nent = 0;
  for (int l = 0; l < 3; ++l) {
    float* P = reinterpret_cast<float*>(sb + p.P[l]);
    w.l[l] = {A_[l], B_[l][0], B_[l][1], P, R64[l], N64[l], nblk};
    nblk += (R64[l] / 64) * (N64[l] / 64) * p.S;
    f.l[l] = {P, R64[l], N64[l], R[l], Nn[l], nent, goff[l]};
    nent += R[l] * Nn[l];
  }
  w.steps = p.steps; w.chunk = p.chunk; w.S = p.S;
  hipLaunchKernelGGL(pg_wgrad_k<Md>, dim3(nblk), dim3(256), 0, st, w);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  f.S = p.S; f.nent = nent; f.nred = (nent + kFinThr - 1) / kFinThr;
  f.col = a.col; f.nwg = p.nwg; f.width = p.AK + p.H2 + p.H1; f.AK = p.AK; f.H2 = p.H2; f.Ap = m.Ap;
  f.boff[0] = gb3; f.boff[1] = gb2; f.boff[2] = gb1;
  f.terms = a.terms; f.M = M; f.c_v = c_v; f.c_h = c_h; f.loss = loss_out; f.grads = grads;
  f.adam = adam ? *adam : AdamStep{};
  const int ncol = (f.width + kColUnits - 1) / kColUnits;
  hipLaunchKernelGGL(pg_finish_k, dim3(f.nred + ncol + 1), dim3(kFinThr), 0, st, f);
  return hipGetLastError();
}

}  // namespace

bool pg_fused_supported(const MlpParams& m) {
  return with_net(m, [](auto) { return hipSuccess; }) == hipSuccess;
}

size_t pg_fused_bytes(const MlpParams& m, int M) { return plan_of(m, M).bytes; }

hipError_t launch_pg_fused(const MlpParams& m, const void* d_weights, const size_t off[6], int T,
                           const float* obs, const uint8_t* act, const float* logp_old,
                           const double* adv, const double* ret, int M, uint64_t seed, float clip,
                           float c_v, float c_h, int reinforce, void* scratch, double* loss_out,
                           float* grads, const AdamStep* adam, int64_t* idx_out, uint32_t* err,
                           hipStream_t st) {
  return with_net(m, [&](auto n) -> hipError_t {
    return run<decltype(n)>(m, d_weights, off, T, obs, act, logp_old, adv, ret, M, seed, clip, c_v,
                            c_h, reinforce, scratch, loss_out, grads, adam, idx_out, err, st);
  });
}

}  // namespace bsim
