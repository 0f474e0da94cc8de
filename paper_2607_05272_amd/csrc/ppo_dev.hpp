// ppo_dev.hpp -- what the kernels of the policy-gradient minibatch share (paper Sec. 4.3): the
// two operand modes, the hidden layers' GELU and its derivative, and one sample's policy term.
#pragma once
#include "devmath.hpp"
#include "params.hpp"

namespace bsim {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ float bf16_round(float f) { return bf16_to_f32(bf16_bits(f)); }
__device__ __forceinline__ float gelu_exact(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// Phi(z), the standard normal distribution, and GELU'(z) = Phi(z) + z phi(z) from one
// exponential. With t = |z|, Phi(-t) = exp(-t^2 / 2) g(t) where g(t) = erfcx(t / sqrt 2) / 2 is
// smooth: 1/2 plus w times a polynomial of degree 6 in w = (t/4) / (1 + t/4), fitted for the
// least maximum of the error of t exp(-t^2/2) g (9.5e-10 before rounding). Against 64 bits over
// [-9, 9] and over normal z, z Phi(z) is off by 5.7e-8 and 1.8e-8 (root mean square; 0.5 z
// (1 + erf) with a correctly rounded erf: 6.4e-8 and 1.9e-8) and GELU' by 2.3e-8 and 2.7e-8
// (2.4e-8 and 2.6e-8). About 22 instructions, where erff and expf take about 90.
__device__ __forceinline__ void gelu_parts(float z, float& Phi, float& grad) {
  // past 20 the tail is 0 in fp32; infinities then give what the definition does
  const float t = fminf(fabsf(z), 20.0f);
  const float w = (0.25f * t) * __builtin_amdgcn_rcpf(fmaf(0.25f, t, 1.0f));
  float g = fmaf(0.07000315189361572f, w, -0.2689400315284729f);
  g = fmaf(g, w, 0.12449410557746887f);
  g = fmaf(g, w, 0.8685218095779419f);
  g = fmaf(g, w, -2.106220006942749f);
  g = fmaf(g, w, 2.404217004776001f);
  g = fmaf(g, w, -1.595768928527832f);
  g = fmaf(g, w, 0.5f);
  const float E = __builtin_amdgcn_exp2f((t * t) * -0.72134752044448170f);   // exp(-t^2 / 2)
  const float tail = E * g;
  Phi = z > 0.0f ? 1.0f - tail : tail;
  grad = fmaf(z, E * 0.39894228040143268f, Phi);
}

// bf16(gelu_exact(z)), the hidden activation in bf16 mode, and GELU'(z). z Phi(z) of gelu_parts and
// gelu_exact differ by at most 3e-7 |z|, so both round to the same bf16 value unless a rounding
// boundary lies within that distance; only then (one activation in some thousands) is
// gelu_exact evaluated. The forward thus keeps the very activations of an erff evaluation:
// a clipped surrogate has a jump at the clip range's edges, and an activation rounded the other
// way moves samples across it.
__device__ __noinline__ f32x4 gelu_exact4(f32x4 z) {
#pragma unroll 1
  for (int i = 0; i < 4; ++i) z = f32x4{z[1], z[2], z[3], gelu_exact(z[0])};
  return z;
}
__device__ __forceinline__ u32x2 gelu_bf16(f32x4 z, f32x4& grad) {
  uint32_t w[4];
  bool near = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float Phi, g;
    gelu_parts(z[i], Phi, g);
    grad[i] = g;
    const float f = z[i] * Phi, d = 3e-7f * fabsf(z[i]);
    w[i] = pack_bf16_pair(f - d, f + d);
    near = near || (w[i] & 0xffffu) != w[i] >> 16;
  }
  u32x2 h{(w[0] & 0xffffu) | (w[1] << 16), (w[2] & 0xffffu) | (w[3] << 16)};
  if (__ballot(near) != 0ull) {   // every lane's four: both forms agree where none is near
    const f32x4 e = gelu_exact4(z);
    h = u32x2{pack_bf16_pair(e[0], e[1]), pack_bf16_pair(e[2], e[3])};
  }
  return h;
}

// Operand modes. Both MFMA shapes take, per lane l, the row (A) or column (B) l % 16 and a run
// of consecutive k (8 bf16 from k = 8 (l / 16), or one fp32 at k = l / 16): every operand
// array is stored k-contiguous, [row][k]. Their 16 x 16 results share one layout: lane l holds
// column l % 16, rows 4 (l / 16) .. + 3.
struct Bf16Mode {
  typedef uint16_t T;
  typedef bf16x8 frag;
  static constexpr int KS = 32, KL = 8, SPLIT = 2, PAD = 8;
  __device__ static int koff(int lane) { return (lane >> 4) * 8; }
  __device__ static frag load(const T* p) { return *reinterpret_cast<const bf16x8*>(p); }
  __device__ static f32x4 mfma(frag a, frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  __device__ static T act(float v) { return bf16_bits(v); }     // activation (already rounded)
  __device__ static float actf(float v) { return bf16_round(v); }
  __device__ static void split(float v, T& hi, T& lo) {
    hi = bf16_bits(v);
    lo = bf16_bits(v - bf16_to_f32(hi));
  }
  __device__ static float value(T v) { return bf16_to_f32(v); }
  // four values rounded to the operand type, and one of them
  typedef u32x2 four;
  // hidden activations of four z and their GELU'
  __device__ static four hidden(f32x4 z, f32x4& grad) { return gelu_bf16(z, grad); }
  __device__ static four pack(const float (&v)[4]) {
    return four{pack_bf16_pair(v[0], v[1]), pack_bf16_pair(v[2], v[3])};
  }
  __device__ static T get(four p, int i) { return (T)(i & 1 ? p[i >> 1] >> 16 : p[i >> 1]); }
};

struct F32Mode {
  typedef float T;
  typedef float frag;
  static constexpr int KS = 4, KL = 1, SPLIT = 1, PAD = 4;
  __device__ static int koff(int lane) { return lane >> 4; }
  __device__ static frag load(const T* p) { return *p; }
  __device__ static f32x4 mfma(frag a, frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static T act(float v) { return v; }
  __device__ static float actf(float v) { return v; }
  __device__ static void split(float v, T& hi, T& lo) { hi = v; lo = 0.f; }
  __device__ static float value(T v) { return v; }
  typedef f32x4 four;
  __device__ static four hidden(f32x4 z, f32x4& grad) {
    four h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = gelu_exact(z[i]);
      grad[i] = gelu_grad(z[i]);
    }
    return h;
  }
  __device__ static four pack(const float (&v)[4]) { return four{v[0], v[1], v[2], v[3]}; }
  __device__ static T get(four p, int i) { return p[i]; }
};

// The taken action's policy term and its derivative with respect to the action's
// log-probability: the clipped surrogate -min(rho A, clip(rho, 1 - eps, 1 + eps) A) with
// rho = exp(logp - logp_old), or (reinforce) -A logp with the advantage held constant.
__device__ __forceinline__ void policy_term(int reinforce, float clip, float logp, float logp_old,
                                            float adv, float invM, float& dlogp, float& pterm) {
  if (reinforce) {
    dlogp = -adv * invM;
    pterm = -adv * logp;
    return;
  }
  const float rho = expf(logp - logp_old);
  const float lo = 1.0f - clip, hi = 1.0f + clip;
  const float rc = fminf(fmaxf(rho, lo), hi);
  const float s1 = rho * adv, s2 = rc * adv;
  const float g_rho = s1 <= s2 ? adv : ((rho > lo && rho < hi) ? adv : 0.0f);
  dlogp = -g_rho * rho * invM;
  pterm = -fminf(s1, s2);
}

}  // namespace
}  // namespace bsim
