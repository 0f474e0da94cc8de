// train_dev.hpp -- one parameter's Adam step (Kingma & Ba 2015, Algorithm 1) and its place in
// the policy's weight buffer, shared by the Adam kernel and the launches that finish a gradient.
#pragma once
#include "devmath.hpp"
#include "params.hpp"

namespace bsim {
namespace {

// the parameter after the step; m and v are updated
__device__ __forceinline__ float adam_param(float p, float g, float& m, float& v, float lr,
                                            float b1, float b2, float eps, float bc1, float bc2) {
  m = b1 * m + (1.0f - b1) * g;
  v = b2 * v + (1.0f - b2) * (g * g);
  const float mhat = m / bc1, vhat = v / bc2;
  return p - lr * mhat / (sqrtf(vhat) + eps);
}

// segment of parameter i, by a short scan of the segment starts
__device__ __forceinline__ int seg_of(const Segs& s, size_t i) {
  int k = 0;
#pragma unroll
  for (int j = 1; j < kMaxSegs; ++j)
    if (j < s.n && i >= s.poff[j]) k = j;
  return k;
}

// parameter i's value into the weight buffer
__device__ __forceinline__ void export_param(const Segs& s, int bf16, unsigned char* w, size_t i,
                                             float p) {
  const int k = seg_of(s, i);
  const size_t j = i - s.poff[k];
  if (s.matrix[k] && bf16) reinterpret_cast<uint16_t*>(w + s.woff[k])[j] = bf16_bits(p);
  else reinterpret_cast<float*>(w + s.woff[k])[j] = p;
}

// Gradient i is done: written, or (a.p != NULL) used for parameter i's step.
__device__ __forceinline__ void finish_param(const AdamStep& a, float* grads, size_t i, float g) {
  if (!a.p) {
    grads[i] = g;
    return;
  }
  float m = a.m[i], v = a.v[i];
  const float p = adam_param(a.p[i], g, m, v, a.lr, a.b1, a.b2, a.eps, a.bc1, a.bc2);
  a.m[i] = m;
  a.v[i] = v;
  a.p[i] = p;
  export_param(a.seg, a.bf16, a.w, i, p);
}

}  // namespace
}  // namespace bsim
