// attn_kernels.hip -- the attention policy of paper Sec. 4.2, fused with action sampling.
//
// Per environment, fp32 (one lane each, or eight in small batches):
//   tokens    e_g = b_in + sum over the features i of group g of x_i W_in[i,:], the F features
//             split into L contiguous groups of F/L (L = 1 is the plain input projection,
//             L = F one token per state feature);
//   attention q, k, v = e W_qkv + b_qkv; per head h (D/NH columns) softmax-weighted values
//             with scores q.k / sqrt(D/NH); y_g = concat_h o_{g,h} W_o + b_o;
//   pooling   p = mean_g y_g;
//   heads     logits = GELU(p W_p1 + b_p1) W_p2 + b_p2, V = GELU(p W_v1 + b_v1) W_v2 + b_v2.
// The action is then drawn by inverse CDF of the fp32 softmax of the logits with the ACTION
// uniform of (env, step), as for the MLP policy.
//
// The network is tiny (D = 4; about 2k multiply-adds per environment), so it runs as plain
// SIMT code: every weight is read at a wave-uniform address (scalar loads through the
// scalar cache), the per-environment state stays in registers, and the observation columns
// obs[f][E] are read coalesced.
#include "ppo_dev.hpp"
#include "train_dev.hpp"

namespace bsim {
namespace {

constexpr int kD = 4;          // embedding width
constexpr int kBlock = 256;

// Scores are kept in base-2 units: the queries carry the factor log2(e) / sqrt(D/NH), so each
// softmax weight is one exp2 of (score - max).
template <int L, int NH, int A>
__global__ __launch_bounds__(kBlock) void attn_policy_k(AttnParams p, int b0, const float* __restrict__ obs,
                                                        const uint64_t* __restrict__ seedp, uint32_t step,
                                                        uint8_t* __restrict__ act,
                                                        float* __restrict__ logp,
                                                        float* __restrict__ value,
                                                        float* __restrict__ logits) {
  const uint64_t seed = *seedp;   // the episode seed
  constexpr int DH = kD / NH;
  constexpr float kLog2e = 1.4426950408889634f;
  const float qscale = (DH == 1 ? 1.0f : DH == 2 ? 0.70710678118654752f : 0.5f) * kLog2e;
  const int e = (b0 + blockIdx.x) * kBlock + threadIdx.x;
  if (e >= p.E) return;
  const size_t E = (size_t)p.E;
  const int G = p.F / L;

  // tokens
  float tok[L][kD];
#pragma unroll
  for (int g = 0; g < L; ++g) {
#pragma unroll
    for (int d = 0; d < kD; ++d) tok[g][d] = p.b_in[d];
    for (int i = g * G; i < (g + 1) * G; ++i) {
      const float x = obs[(size_t)i * E + e];
#pragma unroll
      for (int d = 0; d < kD; ++d) tok[g][d] = fmaf(x, p.w_in[i * kD + d], tok[g][d]);
    }
  }
  // queries, keys, values
  float q[L][kD], k[L][kD], v[L][kD];
#pragma unroll
  for (int g = 0; g < L; ++g) {
#pragma unroll
    for (int d = 0; d < kD; ++d) {
      float aq = p.b_qkv[d], ak = p.b_qkv[kD + d], av = p.b_qkv[2 * kD + d];
#pragma unroll
      for (int i = 0; i < kD; ++i) {
        aq = fmaf(tok[g][i], p.w_qkv[i * 3 * kD + d], aq);
        ak = fmaf(tok[g][i], p.w_qkv[i * 3 * kD + kD + d], ak);
        av = fmaf(tok[g][i], p.w_qkv[i * 3 * kD + 2 * kD + d], av);
      }
      q[g][d] = aq * qscale;
      k[g][d] = ak;
      v[g][d] = av;
    }
  }
  // attention, output projection and mean pooling
  float pool[kD] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < L; ++g) {
    float o[kD];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      float sc[L];
      float mx = -INFINITY;
#pragma unroll
      for (int j = 0; j < L; ++j) {
        float dot = 0.f;
#pragma unroll
        for (int t = h * DH; t < (h + 1) * DH; ++t) dot = fmaf(q[g][t], k[j][t], dot);
        sc[j] = dot;
        mx = fmaxf(mx, sc[j]);
      }
      float S = 0.f;
#pragma unroll
      for (int j = 0; j < L; ++j) {
        sc[j] = __builtin_amdgcn_exp2f(sc[j] - mx);
        S += sc[j];
      }
      const float inv = __builtin_amdgcn_rcpf(S);
#pragma unroll
      for (int t = h * DH; t < (h + 1) * DH; ++t) {
        float acc = 0.f;
#pragma unroll
        for (int j = 0; j < L; ++j) acc = fmaf(sc[j], v[j][t], acc);
        o[t] = acc * inv;
      }
    }
#pragma unroll
    for (int d = 0; d < kD; ++d) {
      float y = p.b_o[d];
#pragma unroll
      for (int i = 0; i < kD; ++i) y = fmaf(o[i], p.w_o[i * kD + d], y);
      pool[d] += y;
    }
  }
#pragma unroll
  for (int d = 0; d < kD; ++d) pool[d] *= 1.0f / (float)L;   // L a power of two: exact

  // policy head
  float lg[A];
#pragma unroll
  for (int a = 0; a < A; ++a) lg[a] = p.bp2[a];
  // unrolled so that the scalar weight loads of several units are in flight together
#pragma unroll 8
  for (int j = 0; j < p.Hp; ++j) {
    float z = p.bp1[j];
#pragma unroll
    for (int d = 0; d < kD; ++d) z = fmaf(pool[d], p.wp1[d * p.Hp + j], z);
    const float hj = gelu_exact(z);
    const float* w2 = p.wp2 + (size_t)j * A;
#pragma unroll
    for (int a = 0; a < A; ++a) lg[a] = fmaf(hj, w2[a], lg[a]);
  }
  // value head
  float V = 0.f;
  if (p.value_head) {
    V = p.bv2[0];
#pragma unroll 8
    for (int j = 0; j < p.Hv; ++j) {
      float z = p.bv1[j];
#pragma unroll
      for (int d = 0; d < kD; ++d) z = fmaf(pool[d], p.wv1[d * p.Hv + j], z);
      V = fmaf(gelu_exact(z), p.wv2[j], V);
    }
  }

  // sampling: fp32 max-subtracted softmax, first action whose running sum exceeds u S
  if (act || logp) {
    float mx = lg[0];
#pragma unroll
    for (int a = 1; a < A; ++a) mx = fmaxf(mx, lg[a]);
    float ex[A];
    float S = 0.f;
#pragma unroll
    for (int a = 0; a < A; ++a) {
      ex[a] = expf(lg[a] - mx);
      S += ex[a];
    }
    const u32x4 w = draw(seed, (uint32_t)e, step, P_ACTION, 0, 0);
    const float target = (((float)(w.x >> 9) + 0.5f) * 0x1p-23f) * S;
    float cum = 0.f, la = lg[A - 1];
    int pick = A - 1;
    bool found = false;
#pragma unroll
    for (int a = 0; a < A; ++a) {
      cum += ex[a];
      const bool take = !found && target < cum;
      pick = take ? a : pick;
      la = take ? lg[a] : la;
      found = found || take;
    }
    if (act) act[e] = (uint8_t)pick;
    if (logp) logp[e] = (la - mx) - logf(S);
  }
  if (value && p.value_head) value[e] = V;
  if (logits) {
#pragma unroll
    for (int a = 0; a < A; ++a) logits[(size_t)a * E + e] = lg[a];
    if (p.value_head) logits[(size_t)A * E + e] = V;
  }
}

__device__ __forceinline__ void wave_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same policy with eight lanes per environment, for batches that leave most SIMDs without a wave
// at one lane each: lane g holds token g, every eighth unit of the heads and every eighth output
// (the value is output A). Every sum is taken by one lane in the one-lane kernel's order, from
// operands that the lanes pass through LDS, so the results are its bits. One wave per workgroup, so
// that no barrier is needed; a head's units run in chunks of kChunk. Bound by one environment's chain
// (22 us in one lane, most of it the heads' 128 erff; 7.4 us in eight), then by issue: about as
// many instructions per environment as the one-lane kernel, whose weights are scalar loads.
constexpr int kLanes = 8, kEnvs = 64 / kLanes, kChunk = 64;
template <int L, int NH, int A>
__global__ __launch_bounds__(64) void attn_policy8_k(AttnParams p, int b0, const float* __restrict__ obs,
                                                     const uint64_t* __restrict__ seedp, uint32_t step,
                                                     uint8_t* __restrict__ act,
                                                     float* __restrict__ logp,
                                                     float* __restrict__ value,
                                                     float* __restrict__ logits) {
  static_assert(L <= kLanes, "a token per lane");
  constexpr int DH = kD / NH, NO = (A + kLanes) / kLanes;   // outputs per lane, the value among them
  constexpr float kLog2e = 1.4426950408889634f;
  const float qscale = (DH == 1 ? 1.0f : DH == 2 ? 0.70710678118654752f : 0.5f) * kLog2e;
  __shared__ __attribute__((aligned(16))) float kv[kEnvs][kLanes][2 * kD], ys[kEnvs][kLanes][kD];
  __shared__ __attribute__((aligned(16))) float hid[2][kEnvs][kChunk + 4];
  __shared__ float lgs[kEnvs][A + 1], exs[kEnvs][A + 1];
  const int lane = threadIdx.x, el = lane / kLanes, g = lane % kLanes;
  const int e = (b0 + blockIdx.x) * kEnvs + el;
  const bool live = e < p.E;
  const size_t E = (size_t)p.E, ee = live ? e : 0;
  const int G = p.F / L;

  // the lane's token, its query, key and value
  float tok[kD], q[kD];
#pragma unroll
  for (int d = 0; d < kD; ++d) tok[d] = p.b_in[d];
  if (g < L)
    for (int i = g * G; i < (g + 1) * G; ++i) {
      const float x = obs[(size_t)i * E + ee];
#pragma unroll
      for (int d = 0; d < kD; ++d) tok[d] = fmaf(x, p.w_in[i * kD + d], tok[d]);
    }
#pragma unroll
  for (int d = 0; d < kD; ++d) {
    float aq = p.b_qkv[d], ak = p.b_qkv[kD + d], av = p.b_qkv[2 * kD + d];
#pragma unroll
    for (int i = 0; i < kD; ++i) {
      aq = fmaf(tok[i], p.w_qkv[i * 3 * kD + d], aq);
      ak = fmaf(tok[i], p.w_qkv[i * 3 * kD + kD + d], ak);
      av = fmaf(tok[i], p.w_qkv[i * 3 * kD + 2 * kD + d], av);
    }
    q[d] = aq * qscale;
    kv[el][g][d] = ak;
    kv[el][g][kD + d] = av;
  }
  wave_lds();
  // attention and output projection of the lane's token, then the mean over the tokens
  float o[kD];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    float sc[L];
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float dot = 0.f;
#pragma unroll
      for (int t = h * DH; t < (h + 1) * DH; ++t) dot = fmaf(q[t], kv[el][j][t], dot);
      sc[j] = dot;
      mx = fmaxf(mx, sc[j]);
    }
    float S = 0.f;
#pragma unroll
    for (int j = 0; j < L; ++j) {
      sc[j] = __builtin_amdgcn_exp2f(sc[j] - mx);
      S += sc[j];
    }
    const float inv = __builtin_amdgcn_rcpf(S);
#pragma unroll
    for (int t = h * DH; t < (h + 1) * DH; ++t) {
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j < L; ++j) acc = fmaf(sc[j], kv[el][j][kD + t], acc);
      o[t] = acc * inv;
    }
  }
#pragma unroll
  for (int d = 0; d < kD; ++d) {
    float y = p.b_o[d];
#pragma unroll
    for (int i = 0; i < kD; ++i) y = fmaf(o[i], p.w_o[i * kD + d], y);
    ys[el][g][d] = y;
  }
  wave_lds();
  float pool[kD] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < L; ++j)
#pragma unroll
    for (int d = 0; d < kD; ++d) pool[d] += ys[el][j][d];
#pragma unroll
  for (int d = 0; d < kD; ++d) pool[d] *= 1.0f / (float)L;

  // the heads, a chunk of units at a time: the lane's units, then its outputs' sums over the chunk
  float acc[NO];
#pragma unroll
  for (int r = 0; r < NO; ++r) {
    const int a = g + kLanes * r;
    acc[r] = a < A ? p.bp2[a] : a == A && p.value_head ? p.bv2[0] : 0.f;
  }
  auto units = [&](float* h, const float* w1, const float* b1, int n, int c) {
#pragma unroll 4
    for (int u = g; u < kChunk; u += kLanes) {
      const int j = c + u < n ? c + u : n - 1;
      float z = b1[j];
#pragma unroll
      for (int d = 0; d < kD; ++d) z = fmaf(pool[d], w1[d * n + j], z);
      h[u] = gelu_exact(z);
    }
  };
  const int Hv = p.value_head ? p.Hv : 0, Hm = p.Hp > Hv ? p.Hp : Hv;
  for (int c = 0; c < Hm; c += kChunk) {
    wave_lds();
    if (c < p.Hp) units(hid[0][el], p.wp1, p.bp1, p.Hp, c);
    if (c < Hv) units(hid[1][el], p.wv1, p.bv1, Hv, c);
    wave_lds();
#pragma unroll
    for (int r = 0; r < NO; ++r) {
      const int a = g + kLanes * r;
      const bool val = a >= A;
      const int n = a > A ? 0 : (val ? Hv : p.Hp) - c;   // units left (none past the value)
      const float* h = hid[val ? 1 : 0][el];
      const float* w = val ? p.wv2 + c : p.wp2 + (size_t)c * A + a;
      const int sw = val ? 1 : A;
      if (n >= kChunk) {
#pragma unroll 16
        for (int u = 0; u < kChunk; ++u) acc[r] = fmaf(h[u], w[u * sw], acc[r]);
      } else {
        for (int u = 0; u < n; ++u) acc[r] = fmaf(h[u], w[u * sw], acc[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NO; ++r) {
    const int a = g + kLanes * r;
    if (a < A) lgs[el][a] = acc[r];
    if (live && a <= A && logits && (a < A || p.value_head)) logits[(size_t)a * E + e] = acc[r];
    if (live && a == A && value && p.value_head) value[e] = acc[r];
  }
  if (!act && !logp) return;
  // sampling: the exponentials by the lanes, the running sums by the environment's first lane
  wave_lds();
  float mx = lgs[el][0];
#pragma unroll
  for (int a = 1; a < A; ++a) mx = fmaxf(mx, lgs[el][a]);
#pragma unroll
  for (int r = 0; r < NO; ++r) {
    const int a = g + kLanes * r;
    if (a < A) exs[el][a] = expf(acc[r] - mx);
  }
  const u32x4 w = draw(*seedp, (uint32_t)e, step, P_ACTION, 0, 0);
  wave_lds();
  if (g != 0 || !live) return;
  float S = 0.f;
#pragma unroll
  for (int a = 0; a < A; ++a) S += exs[el][a];
  const float target = (((float)(w.x >> 9) + 0.5f) * 0x1p-23f) * S;
  float cum = 0.f;
  int pick = A - 1;
  bool found = false;
#pragma unroll
  for (int a = 0; a < A; ++a) {
    cum += exs[el][a];
    const bool take = !found && target < cum;
    pick = take ? a : pick;
    found = found || take;
  }
  if (act) act[e] = (uint8_t)pick;
  if (logp) logp[e] = (lgs[el][pick] - mx) - logf(S);
}

// Batches that take eight lanes per environment: up to five rounds of one wave per SIMD (us, against
// one lane: 256 environments 7.4, 22.0; 16384 11.7, 22.8; 40000 21.0, 23.1; 50000 23.8, 23.4; with
// 24 actions 40000 24.5, 40.7; with 256-unit heads 40000 66.5, 72.0).
constexpr int kWideE = 40960;

template <int L, int NH, int A>
hipError_t run_attn(const AttnParams& p, const float* obs, const uint64_t* seed, uint32_t step,
                    uint8_t* act, float* logp, float* value, float* logits, EnvPart part, hipStream_t st) {
  if (p.E <= kWideE) {
    if (part.e0 % kEnvs != 0) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((part.n + kEnvs - 1) / kEnvs)), block(64);
    hipLaunchKernelGGL((attn_policy8_k<L, NH, A>), grid, block, 0, st, p, part.e0 / kEnvs, obs, seed,
                       step, act, logp, value, logits);
    return hipGetLastError();
  }
  if (part.e0 % kBlock != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((part.n + kBlock - 1) / kBlock)), block(kBlock);
  hipLaunchKernelGGL((attn_policy_k<L, NH, A>), grid, block, 0, st, p, part.e0 / kBlock, obs, seed, step, act, logp,
                     value, logits);
  return hipGetLastError();
}

template <int L, int NH>
hipError_t run_attn_a(const AttnParams& p, const float* obs, const uint64_t* seed, uint32_t step,
                      uint8_t* act, float* logp, float* value, float* logits, EnvPart part, hipStream_t st) {
  switch (p.A) {
    case 6: return run_attn<L, NH, 6>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 12: return run_attn<L, NH, 12>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 24: return run_attn<L, NH, 24>(p, obs, seed, step, act, logp, value, logits, part, st);
    default: return hipErrorInvalidValue;
  }
}

template <int L>
hipError_t run_attn_h(const AttnParams& p, const float* obs, const uint64_t* seed, uint32_t step,
                      uint8_t* act, float* logp, float* value, float* logits, EnvPart part, hipStream_t st) {
  switch (p.NH) {
    case 1: return run_attn_a<L, 1>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 2: return run_attn_a<L, 2>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 4: return run_attn_a<L, 4>(p, obs, seed, step, act, logp, value, logits, part, st);
    default: return hipErrorInvalidValue;
  }
}

// ---- gradient of one minibatch (Sec. 4.3 losses through the Sec. 4.2 network) --------------
// Eight lanes per sample m, lane g of them holding token g (idle where g >= L) and every eighth
// unit of the heads: the (t, env) index drawn like the MLP minibatch's, the forward in fp32, the
// loss gradient with respect to the logits and V, then the chain rule backwards. The pooled
// vector's gradient dp reaches every token's output equally (dy_g = dp / L), so
// dW_o = (sum_g o_g)^T dy, do_g = dy W_o^T is the same for every token and so is
// da_{gj} = do . v_j per head. What a query's lane needs of the other tokens (keys and values, and
// in the backward the softmax weights and score gradients of their queries) it reads from the
// sample's slice of LDS; the eight lanes are part of one wave, so no barrier is needed for it.
//
// A workgroup takes kSamples samples. The heads run in chunks of kUnits units staged in LDS; in
// the backward the chunk's activations and gradients dz go to LDS and each thread sums its
// parameters' terms over the workgroup's samples, while the attention's parameters are summed
// over the wave's lanes. Each workgroup writes one row of partial sums [P]; attn_finish_k adds
// the rows in a fixed order. Bound by the chain of one sample's layers at one wave per SIMD:
// 8192 samples of the 8-token, 2-head, 64-unit network take 20 us and the sums with Adam's step 4
// (one lane per sample, on an eighth of the SIMDs, with every per-sample term through memory:
// 159 us and, in four launches, 27).
struct AttnGradArgs {
  AttnParams p;
  int T, M, reinforce;
  const float* obs;          // [T(+1)][F][E]
  const uint8_t* act;        // [T][E]
  const float* logp_old;     // [T][E] (PPO)
  const double* adv;         // [T][E]
  const double* ret;         // [T][E]
  uint64_t seed;
  float clip, c_v, c_h;
  float* part;               // [workgroups][P] partial sums of the gradient
  double* terms;             // [workgroups][3] policy, value, entropy sums
  int64_t* idx_out;          // optional [M]
  uint32_t* err;
  int off[14];               // start of each parameter array in the gradient vector
  int P;
};

constexpr int kSamples = 32, kUnits = 64, kUStride = kUnits + 8;   // rows 8 banks apart
constexpr int kGradThr = 8 * kSamples;
// a sample's slice: keys and values of its tokens, and one head's [query][key] of weights and
// score gradients with the queries they go with
struct AttnSlice {
  float kv[8][8];
  float a[8][9], ds[8][9];
  float q[8][4];
};
template <int A>
struct HeadChunk {           // one chunk of a head's weights (the value head: A = 1)
  float w1[kD][kUnits], b1[kUnits], w2[kUnits][A];
};
template <int A>
struct AttnGradLds {
  AttnSlice sl[kSamples];
  HeadChunk<A> pol;
  HeadChunk<1> val;
  float h[kSamples][kUStride], dz[kSamples][kUStride];   // the backward's chunk
  float dl[kSamples][A], dV[kSamples], pool[kSamples][kD];
  double terms[kSamples][3];
};

// Sums by DPP moves within rows of 16 lanes (two samples): over a sample's 8 lanes (quads, then
// the other quad by a half-row mirror), and with the other sample's lane of the same part (a
// rotation by 8); every lane that shares a sum gets the same bits.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float sum8(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  return v + dpp_f<0x141>(v);
}
__device__ __forceinline__ float sum_pair(float v) { return v + dpp_f<0x128>(v); }

// Units j0 .. j0 + kUnits - 1 of a head (zero past its n units) into LDS, by the workgroup.
template <int A>
__device__ __forceinline__ void stage_head(HeadChunk<A>& c, const float* w1, const float* b1,
                                           const float* w2, int n, int j0) {
  for (int q = threadIdx.x; q < kUnits * (kD + 1 + A); q += kGradThr) {
    const int r = q / kUnits, u = q % kUnits;
    if (r < kD) {
      c.w1[r][u] = j0 + u < n ? w1[r * n + j0 + u] : 0.f;
    } else if (r == kD) {
      c.b1[u] = j0 + u < n ? b1[j0 + u] : 0.f;
    } else {
      const int e = (r - kD - 1) * kUnits + u;   // w2's rows of this chunk are contiguous
      (&c.w2[0][0])[e] = j0 * A + e < n * A ? w2[j0 * A + e] : 0.f;
    }
  }
}

template <int L, int NH, int A>
__global__ __launch_bounds__(kGradThr) void attn_grad_k(AttnGradArgs g) {
  constexpr int D = kD, DH = D / NH;
  const float rs = DH == 1 ? 1.0f : DH == 2 ? 0.70710678118654752f : 0.5f;  // 1 / sqrt(DH)
  __shared__ AttnGradLds<A> S;
  const int tid = threadIdx.x, lane = tid & 63, sl = tid >> 3, gg = tid & 7;
  const int m = blockIdx.x * kSamples + sl;
  const AttnParams& p = g.p;
  const size_t E = (size_t)p.E;
  const int G = p.F / L;
  const bool tokn = gg < L;          // the lane holds a token
  float* part = g.part + (size_t)blockIdx.x * g.P;

  // the heads' first chunks, while the sample is fetched
  stage_head<A>(S.pol, p.wp1, p.bp1, p.wp2, p.Hp, 0);
  stage_head<1>(S.val, p.wv1, p.bv1, p.wv2, p.Hv, 0);

  // the sample: past M it is computed with a zero observation and contributes nothing, and so does
  // one whose stored action is invalid (flagged)
  long long ix = 0;
  if (m < g.M) {
    const u32x4 w = draw(g.seed, (uint32_t)m, 0xFFFFFFFDu, P_MINIBATCH, 0, 0);
    ix = (long long)(unit(w.x, w.y) * ((double)g.T * (double)p.E));
    if (ix > (long long)g.T * p.E - 1) ix = (long long)g.T * p.E - 1;
    if (gg == 0 && g.idx_out) g.idx_out[m] = ix;
  }
  const int t = (int)ix / p.E, e = (int)ix - t * p.E;   // T E < 2^31 (checked by the host)
  const size_t ti = (size_t)ix;
  const float* xo = g.obs + (size_t)t * p.F * E + e;
  const int a_act = g.act[ti];
  const float adv = (float)g.adv[ti], ret = (float)g.ret[ti];
  const float lold = g.reinforce ? 0.f : g.logp_old[ti];
  const bool bad = m < g.M && a_act >= A;
  if (bad && gg == 0) atomicOr(g.err, ERR_ACTION);
  const bool on = m < g.M && !bad;

  // forward: the lane's token, its query, key and value
  float tok[D];
#pragma unroll
  for (int d = 0; d < D; ++d) tok[d] = p.b_in[d];
  if (tokn)
    for (int i = gg * G; i < (gg + 1) * G; ++i) {
      const float x = on ? xo[(size_t)i * E] : 0.f;
#pragma unroll
      for (int d = 0; d < D; ++d) tok[d] = fmaf(x, p.w_in[i * D + d], tok[d]);
    }
  float q[D], k[D], v[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    float aq = p.b_qkv[d], ak = p.b_qkv[D + d], av = p.b_qkv[2 * D + d];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      aq = fmaf(tok[i], p.w_qkv[i * 3 * D + d], aq);
      ak = fmaf(tok[i], p.w_qkv[i * 3 * D + D + d], ak);
      av = fmaf(tok[i], p.w_qkv[i * 3 * D + 2 * D + d], av);
    }
    q[d] = aq; k[d] = ak; v[d] = av;
  }
  AttnSlice& X = S.sl[sl];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    X.kv[gg][d] = k[d];
    X.kv[gg][D + d] = v[d];
    X.q[gg][d] = q[d];
  }
  wave_lds();
  float att[NH][L];   // softmax weights of the lane's query
  float osum[D];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    float mx = -INFINITY, s = 0.f, o[DH];
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float dot = 0.f;
#pragma unroll
      for (int x = 0; x < DH; ++x) dot = fmaf(q[h * DH + x], X.kv[j][h * DH + x], dot);
      att[h][j] = dot * rs;
      mx = fmaxf(mx, att[h][j]);
    }
#pragma unroll
    for (int j = 0; j < L; ++j) {
      att[h][j] = expf(att[h][j] - mx);
      s += att[h][j];
    }
    const float inv = tokn ? 1.0f / s : 0.f;
#pragma unroll
    for (int x = 0; x < DH; ++x) o[x] = 0.f;
#pragma unroll
    for (int j = 0; j < L; ++j) {
      att[h][j] *= inv;   // zero in lanes without a token
#pragma unroll
      for (int x = 0; x < DH; ++x) o[x] = fmaf(att[h][j], X.kv[j][D + h * DH + x], o[x]);
    }
#pragma unroll
    for (int x = 0; x < DH; ++x) osum[h * DH + x] = sum8(o[x]);
  }
  float pool[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    float y = 0.f;
#pragma unroll
    for (int i = 0; i < D; ++i) y = fmaf(osum[i], p.w_o[i * D + d], y);
    pool[d] = y * (1.0f / (float)L) + p.b_o[d];
  }
  // heads forward: the lane's units of every chunk, then the sample's sums
  float lg[A], V = 0.f;
#pragma unroll
  for (int a = 0; a < A; ++a) lg[a] = 0.f;
  const int npol = (p.Hp + kUnits - 1) / kUnits, nval = (p.Hv + kUnits - 1) / kUnits;
  for (int c = 0; c < npol; ++c) {
    if (c > 0) {
      __syncthreads();
      stage_head<A>(S.pol, p.wp1, p.bp1, p.wp2, p.Hp, c * kUnits);
    }
    __syncthreads();
#pragma unroll 2
    for (int u = gg; u < kUnits; u += 8) {
      float z = S.pol.b1[u], Phi, gr;
#pragma unroll
      for (int d = 0; d < D; ++d) z = fmaf(pool[d], S.pol.w1[d][u], z);
      gelu_parts(z, Phi, gr);
      const float hj = z * Phi;
#pragma unroll
      for (int a = 0; a < A; ++a) lg[a] = fmaf(hj, S.pol.w2[u][a], lg[a]);
    }
  }
  for (int c = 0; c < nval; ++c) {
    if (c > 0) {
      __syncthreads();
      stage_head<1>(S.val, p.wv1, p.bv1, p.wv2, p.Hv, c * kUnits);
      __syncthreads();
    }
#pragma unroll 2
    for (int u = gg; u < kUnits; u += 8) {
      float z = S.val.b1[u], Phi, gr;
#pragma unroll
      for (int d = 0; d < D; ++d) z = fmaf(pool[d], S.val.w1[d][u], z);
      gelu_parts(z, Phi, gr);
      V = fmaf(z * Phi, S.val.w2[u][0], V);
    }
  }
#pragma unroll
  for (int a = 0; a < A; ++a) lg[a] = sum8(lg[a]) + p.bp2[a];
  V = sum8(V) + p.bv2[0];

  // loss terms and their gradient with respect to the logits and V (every lane of the sample)
  float mx = lg[0];
#pragma unroll
  for (int a = 1; a < A; ++a) mx = fmaxf(mx, lg[a]);
  float s = 0.f;
#pragma unroll
  for (int a = 0; a < A; ++a) s += expf(lg[a] - mx);
  const float lS = logf(s);
  float pa[A], H = 0.f, l_act = lg[0];
#pragma unroll
  for (int a = 0; a < A; ++a) {
    const float lp = (lg[a] - mx) - lS;
    pa[a] = expf(lp);
    H -= pa[a] * lp;
    l_act = a == a_act ? lg[a] : l_act;
  }
  const float logp = (l_act - mx) - lS;
  const float invM = 1.0f / (float)g.M;
  float dlogp, pterm;
  policy_term(g.reinforce, g.clip, logp, lold, adv, invM, dlogp, pterm);
  float dl[A];
#pragma unroll
  for (int a = 0; a < A; ++a) {
    const float lp = (lg[a] - mx) - lS;
    dl[a] = on ? -dlogp * pa[a] + g.c_h * invM * pa[a] * (lp + H) + (a == a_act ? dlogp : 0.0f)
               : 0.f;
  }
  const float dV = p.value_head && on ? 2.0f * g.c_v * (V - ret) * invM : 0.0f;
  if (gg == 0) {
#pragma unroll
    for (int a = 0; a < A; ++a) S.dl[sl][a] = dl[a];
    S.dV[sl] = dV;
#pragma unroll
    for (int d = 0; d < D; ++d) S.pool[sl][d] = pool[d];
    S.terms[sl][0] = on ? (double)pterm : 0.0;
    S.terms[sl][1] = on ? (double)(V - ret) * (double)(V - ret) : 0.0;
    S.terms[sl][2] = on ? (double)H : 0.0;
  }

  // heads backward, a chunk at a time
  float dp[D] = {0.f, 0.f, 0.f, 0.f};
  const int pu = tid & 63, pr = tid >> 6;   // the thread's unit and row in the parameter sums
  for (int c = 0; c < npol; ++c) {
    if (npol > 1) {
      __syncthreads();
      stage_head<A>(S.pol, p.wp1, p.bp1, p.wp2, p.Hp, c * kUnits);
      __syncthreads();
    }
#pragma unroll 2
    for (int u = gg; u < kUnits; u += 8) {
      float z = S.pol.b1[u], Phi, gr, dh = 0.f;
#pragma unroll
      for (int d = 0; d < D; ++d) z = fmaf(pool[d], S.pol.w1[d][u], z);
      gelu_parts(z, Phi, gr);
#pragma unroll
      for (int a = 0; a < A; ++a) dh = fmaf(dl[a], S.pol.w2[u][a], dh);
      const float dz = dh * gr;
      S.h[sl][u] = z * Phi;
      S.dz[sl][u] = dz;
#pragma unroll
      for (int d = 0; d < D; ++d) dp[d] = fmaf(dz, S.pol.w1[d][u], dp[d]);
    }
    __syncthreads();
    const int j = c * kUnits + pu;
    float s1 = 0.f, sb = 0.f, s2[(A + 3) / 4];
#pragma unroll
    for (int i = 0; i < (A + 3) / 4; ++i) s2[i] = 0.f;
#pragma unroll 4
    for (int x = 0; x < kSamples; ++x) {
      const float dz = S.dz[x][pu], hj = S.h[x][pu];
      s1 = fmaf(S.pool[x][pr], dz, s1);
      sb += dz;
#pragma unroll
      for (int i = 0; i < (A + 3) / 4; ++i)
        if (pr + 4 * i < A) s2[i] = fmaf(hj, S.dl[x][pr + 4 * i], s2[i]);
    }
    if (j < p.Hp) {
      part[g.off[6] + pr * p.Hp + j] = s1;
      if (pr == 0) part[g.off[7] + j] = sb;
#pragma unroll
      for (int i = 0; i < (A + 3) / 4; ++i)
        if (pr + 4 * i < A) part[g.off[8] + j * A + pr + 4 * i] = s2[i];
    }
    __syncthreads();
  }
  for (int c = 0; c < nval; ++c) {
    if (nval > 1) {
      stage_head<1>(S.val, p.wv1, p.bv1, p.wv2, p.Hv, c * kUnits);
      __syncthreads();
    }
#pragma unroll 2
    for (int u = gg; u < kUnits; u += 8) {
      float z = S.val.b1[u], Phi, gr;
#pragma unroll
      for (int d = 0; d < D; ++d) z = fmaf(pool[d], S.val.w1[d][u], z);
      gelu_parts(z, Phi, gr);
      const float dz = dV * S.val.w2[u][0] * gr;
      S.h[sl][u] = z * Phi;
      S.dz[sl][u] = dz;
#pragma unroll
      for (int d = 0; d < D; ++d) dp[d] = fmaf(dz, S.val.w1[d][u], dp[d]);
    }
    __syncthreads();
    const int j = c * kUnits + pu;
    float s1 = 0.f, sb = 0.f, s2 = 0.f;
#pragma unroll 4
    for (int x = 0; x < kSamples; ++x) {
      const float dz = S.dz[x][pu];
      s1 = fmaf(S.pool[x][pr], dz, s1);
      sb += dz;
      s2 = fmaf(S.h[x][pu], S.dV[x], s2);
    }
    if (j < p.Hv) {
      part[g.off[10] + pr * p.Hv + j] = s1;
      if (pr == 0) part[g.off[11] + j] = sb;
      if (pr == 1) part[g.off[12] + j] = s2;
    }
    __syncthreads();
  }
  // biases of the heads' outputs and the loss terms: sums over the samples in order
  if (tid < A) {
    float x = 0.f;
    for (int i = 0; i < kSamples; ++i) x += S.dl[i][tid];
    part[g.off[9] + tid] = x;
  } else if (tid == 64) {
    float x = 0.f;
    for (int i = 0; i < kSamples; ++i) x += S.dV[i];
    part[g.off[13]] = x;
  } else if (tid >= 128 && tid < 131) {
    double x = 0.0;
    for (int i = 0; i < kSamples; ++i) x += S.terms[i][tid - 128];
    g.terms[(size_t)blockIdx.x * 3 + tid - 128] = x;
  }

  // output projection: dy = dp / L for every token
  float dO[D];
#pragma unroll
  for (int d = 0; d < D; ++d) dp[d] = sum8(dp[d]);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    float acc = 0.f;
#pragma unroll
    for (int d = 0; d < D; ++d) acc = fmaf(dp[d] * (1.0f / (float)L), p.w_o[i * D + d], acc);
    dO[i] = acc;
  }
  // attention backward, head by head: the query's score gradients, then each key's and value's
  // share of all queries'
  float dq[D], dk[D], dv[D];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    float sd = 0.f, da[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float acc = 0.f;
#pragma unroll
      for (int x = 0; x < DH; ++x) acc = fmaf(dO[h * DH + x], X.kv[j][D + h * DH + x], acc);
      da[j] = acc;
      sd = fmaf(att[h][j], acc, sd);
    }
    float aq[DH];
#pragma unroll
    for (int x = 0; x < DH; ++x) aq[x] = 0.f;
    wave_lds();   // the previous head's reads are done
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const float ds = att[h][j] * (da[j] - sd) * rs;   // zero in lanes without a token
      X.a[gg][j] = att[h][j];
      X.ds[gg][j] = ds;
#pragma unroll
      for (int x = 0; x < DH; ++x) aq[x] = fmaf(ds, X.kv[j][h * DH + x], aq[x]);
    }
    wave_lds();
    float cs = 0.f, ak[DH];
#pragma unroll
    for (int x = 0; x < DH; ++x) ak[x] = 0.f;
    const int me = tokn ? gg : 0;   // lanes without a token read column 0 and drop it
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const float ds = X.ds[j][me];
      cs += X.a[j][me];
#pragma unroll
      for (int x = 0; x < DH; ++x) ak[x] = fmaf(ds, X.q[j][h * DH + x], ak[x]);
    }
#pragma unroll
    for (int x = 0; x < DH; ++x) {
      dq[h * DH + x] = aq[x];
      dk[h * DH + x] = tokn ? ak[x] : 0.f;
      dv[h * DH + x] = tokn ? cs * dO[h * DH + x] : 0.f;
    }
  }
  // q/k/v projection and the token. The attention's parameters (W_qkv [D][3D], b_qkv, W_o [D][D],
  // b_o, b_in: entries 0 .. kEnt - 1) are summed over rows of 16 lanes, entry n kept by the
  // row's lane n % 16, then over the workgroup's rows through LDS.
  constexpr int kEnt = 84, kRows = kGradThr / 16;
  float* ws = &S.h[0][0];   // [kRows][kEnt], free after the heads
  static_assert(kRows * kEnt <= kSamples * kUStride, "room for the rows' sums");
  float de[D];
#pragma unroll
  for (int i = 0; i < D; ++i) de[i] = 0.f;
  float keep[(kEnt + 15) / 16];
#pragma unroll
  for (int i = 0; i < (kEnt + 15) / 16; ++i) keep[i] = 0.f;
  auto entry = [&](int n, float v) {   // v: the lane's term of entry n
    const float x = sum_pair(sum8(v));
    keep[n >> 4] = (n & 15) == (lane & 15) ? x : keep[n >> 4];
  };
#pragma unroll
  for (int c = 0; c < 3 * D; ++c) {
    const float col = c < D ? dq[c % D] : c < 2 * D ? dk[c % D] : dv[c % D];
    entry(4 * 3 * D + c, col);
#pragma unroll
    for (int i = 0; i < D; ++i) {
      entry(i * 3 * D + c, tok[i] * col);
      de[i] = fmaf(col, p.w_qkv[i * 3 * D + c], de[i]);
    }
  }
  const float own = gg == 0 ? 1.f : 0.f;   // per-sample terms, counted once
#pragma unroll
  for (int i = 0; i < D; ++i)
#pragma unroll
    for (int d = 0; d < D; ++d) entry(60 + i * D + d, own * (osum[i] * (dp[d] * (1.0f / (float)L))));
#pragma unroll
  for (int d = 0; d < D; ++d) {
    entry(76 + d, own * dp[d]);
    entry(80 + d, tokn ? de[d] : 0.f);
  }
  const int row = tid >> 4;
#pragma unroll
  for (int i = 0; i < (kEnt + 15) / 16; ++i) {
    const int n = i * 16 + (lane & 15);
    if (n < kEnt) ws[row * kEnt + n] = keep[i];
  }
  __syncthreads();
  if (tid < kEnt) {
    float x = ws[tid];
#pragma unroll
    for (int r = 1; r < kRows; ++r) x += ws[r * kEnt + tid];
    const int n = tid;
    const int o = n < 48 ? g.off[2] + n : n < 60 ? g.off[3] + n - 48 : n < 76 ? g.off[4] + n - 60
                : n < 80 ? g.off[5] + n - 76 : g.off[1] + n - 80;
    part[o] = x;
  }
  // W_in: feature gg G + r of the lane's token, summed over the samples the same way
  for (int r = 0; r < G; ++r) {
    const float x = tokn && on ? xo[(size_t)(gg * G + r) * E] : 0.f;
    __syncthreads();   // the previous sums are read
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const float y = sum_pair(x * de[d]);
      if ((lane & 8) == 0) ws[(row * 8 + gg) * D + d] = y;
    }
    __syncthreads();
    if (tid < 8 * D && tid / D < L) {
      float y = ws[tid];
#pragma unroll
      for (int w = 1; w < kRows; ++w) y += ws[w * 8 * D + tid];
      part[g.off[0] + ((tid / D) * G + r) * D + tid % D] = y;
    }
  }
}

// The workgroups' partial sums and loss terms added in a fixed order: kFinCols parameters per
// workgroup, part t of them adding rows t, t + kFinParts, ... in order, then the parts in order; the last
// workgroup the loss terms.
struct AttnFinArgs {
  const float* part;
  const double* terms;
  int nwg, P, M;
  float c_v, c_h;
  float* grads;
  double* loss;
  AdamStep adam;   // p NULL: the gradient is written
};
constexpr int kFinThr = 256, kFinCols = 16, kFinParts = kFinThr / kFinCols;
__global__ __launch_bounds__(kFinThr) void attn_finish_k(AttnFinArgs a) {
  const int tid = threadIdx.x;
  if (blockIdx.x < gridDim.x - 1) {
    __shared__ float part[kFinParts][kFinCols + 1];
    const int i = blockIdx.x * kFinCols + tid % kFinCols, t = tid / kFinCols;
    float s = 0.f;
    if (i < a.P) {
#pragma unroll 8
      for (int w = t; w < a.nwg; w += kFinParts) s += a.part[(size_t)w * a.P + i];
    }
    part[t][tid % kFinCols] = s;
    __syncthreads();
    if (t == 0 && i < a.P) {
#pragma unroll
      for (int w = 1; w < kFinParts; ++w) s += part[w][tid];
      finish_param(a.adam, a.grads, (size_t)i, s);
    }
    return;
  }
  __shared__ double dp[3][kFinThr];
  for (int c = 0; c < 3; ++c) {
    double s = 0.0;
    for (int w = tid; w < a.nwg; w += kFinThr) s += a.terms[(size_t)w * 3 + c];
    dp[c][tid] = s;
  }
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

template <int L, int NH, int A>
hipError_t run_grad(const AttnGradArgs& g, hipStream_t st) {
  hipLaunchKernelGGL((attn_grad_k<L, NH, A>), dim3((unsigned)((g.M + kSamples - 1) / kSamples)),
                     dim3(kGradThr), 0, st, g);
  return hipGetLastError();
}
template <int L, int NH>
hipError_t run_grad_a(const AttnGradArgs& g, hipStream_t st) {
  switch (g.p.A) {
    case 6: return run_grad<L, NH, 6>(g, st);
    case 12: return run_grad<L, NH, 12>(g, st);
    case 24: return run_grad<L, NH, 24>(g, st);
    default: return hipErrorInvalidValue;
  }
}
template <int L>
hipError_t run_grad_h(const AttnGradArgs& g, hipStream_t st) {
  switch (g.p.NH) {
    case 1: return run_grad_a<L, 1>(g, st);
    case 2: return run_grad_a<L, 2>(g, st);
    case 4: return run_grad_a<L, 4>(g, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int attn_param_count(const AttnParams& p, int off[14]) {
  const int D = p.D, n[14] = {p.F * D, D, D * 3 * D, 3 * D, D * D, D, D * p.Hp, p.Hp,
                              p.Hp * p.A, p.A, D * p.Hv, p.Hv, p.Hv, 1};
  int acc = 0;
  for (int i = 0; i < 14; ++i) {
    if (off) off[i] = acc;
    acc += n[i];
  }
  return acc;
}

// a row of partial sums and the loss terms per workgroup
static int grad_workgroups(int M) { return (M + kSamples - 1) / kSamples; }
size_t attn_grad_scratch_bytes(const AttnParams& p, int M) {
  return (size_t)grad_workgroups(M) *
         ((size_t)attn_param_count(p, nullptr) * sizeof(float) + 3 * sizeof(double));
}
size_t attn_stated_bytes(const AttnParams& p, int M) {
  return (size_t)attn_param_count(p, nullptr) * M * sizeof(float) + (size_t)M * 3 * sizeof(double);
}

hipError_t launch_attn_grad(const AttnParams& p, int T, const float* obs, const uint8_t* act,
                            const float* logp_old, const double* adv, const double* ret, int M,
                            uint64_t seed, float clip, float c_v, float c_h, int reinforce,
                            void* scratch, double* loss_out, float* grads, const AdamStep* adam,
                            int64_t* idx_out, uint32_t* err, hipStream_t st) {
  if (!attn_shape_supported(p) || M < 1) return hipErrorInvalidValue;
  AttnGradArgs g;
  g.p = p; g.T = T; g.M = M; g.reinforce = reinforce;
  g.obs = obs; g.act = act; g.logp_old = logp_old; g.adv = adv; g.ret = ret;
  g.seed = seed; g.clip = clip; g.c_v = c_v; g.c_h = c_h;
  g.P = attn_param_count(p, g.off);
  // the loss terms (8-byte aligned at the start), then the partial sums
  const int nwg = grad_workgroups(M);
  g.terms = static_cast<double*>(scratch);
  g.part = reinterpret_cast<float*>(g.terms + (size_t)nwg * 3);
  g.idx_out = idx_out; g.err = err;
  hipError_t e;
  switch (p.L) {
    case 1: e = run_grad_h<1>(g, st); break;
    case 2: e = run_grad_h<2>(g, st); break;
    case 4: e = run_grad_h<4>(g, st); break;
    case 8: e = run_grad_h<8>(g, st); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  AttnFinArgs f{g.part, g.terms, nwg, g.P, M, c_v, c_h, grads, loss_out,
                adam ? *adam : AdamStep{}};
  hipLaunchKernelGGL(attn_finish_k, dim3((unsigned)((g.P + kFinCols - 1) / kFinCols + 1)),
                     dim3(kFinThr), 0, st, f);
  return hipGetLastError();
}

bool attn_shape_supported(const AttnParams& p) {
  const bool L_ok = p.L == 1 || p.L == 2 || p.L == 4 || p.L == 8;
  const bool H_ok = p.NH == 1 || p.NH == 2 || p.NH == 4;
  const bool A_ok = p.A == 6 || p.A == 12 || p.A == 24;
  return L_ok && H_ok && A_ok && p.D == kD && p.F % p.L == 0 && p.Hp >= 1 && p.Hv >= 1;
}

hipError_t launch_attn_policy(const AttnParams& p, const float* obs, const uint64_t* seed, uint32_t step,
                              uint8_t* act, float* logp, float* value, float* logits,
                              EnvPart part, hipStream_t st) {
  if (!attn_shape_supported(p)) return hipErrorInvalidValue;
  switch (p.L) {
    case 1: return run_attn_h<1>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 2: return run_attn_h<2>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 4: return run_attn_h<4>(p, obs, seed, step, act, logp, value, logits, part, st);
    case 8: return run_attn_h<8>(p, obs, seed, step, act, logp, value, logits, part, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bsim
