// gae_kernels.hip -- discounted returns / GAE (paper Sec. 4.3) over a [T][E] trajectory.
//
//   delta_t = (r_t + gamma V_{t+1}) - V_t,  A_t = delta_t + (gamma*lambda) A_{t+1},
//   A_T = 0,  R_t = A_t + V_t,
// backwards in t, in fp64 with V read as fp32 and widened: per environment a chain of one
// multiplication and one addition per step, over 28 bytes of memory traffic per step. Both forms
// below take the steps of an environment in order with the same operations, so their results
// are the same bits.
#include "params.hpp"

namespace bsim {
namespace {

// Large batches: one lane per environment, every row access coalesced. Bound by HBM once enough
// loads are in flight: a lane that loads one row, sums it and stores it waits out a memory
// round trip per step (65536 x 1024: 1080 us, 1.7 TB/s), so the rows of the next kAhead steps
// are loaded while the current ones are summed and stored (345 us, 5.45 TB/s; a plain copy
// reaches 5.2).
constexpr int kAhead = 8;
template <bool HASV>
__global__ __launch_bounds__(64) void gae_stream_k(int T, int E, const double* __restrict__ r,
                                                   const float* __restrict__ v, double gamma,
                                                   double gl, double* __restrict__ adv,
                                                   double* __restrict__ ret) {
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= E) return;
  const size_t sE = (size_t)E;
  double a = 0.0, vn = HASV ? (double)v[(size_t)T * sE + e] : 0.0;
  auto step = [&](size_t i, double rt, double vt) {
    const double delta = (rt + gamma * vn) - vt;
    a = delta + gl * a;
    adv[i] = a;
    ret[i] = a + vt;
    vn = vt;
  };
  int t = T;
  for (; t % kAhead; --t) {
    const size_t i = (size_t)(t - 1) * sE + e;
    step(i, r[i], HASV ? (double)v[i] : 0.0);
  }
  if (t == 0) return;
  double rb[kAhead];
  float vb[kAhead];
  auto load = [&](int hi) {
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const size_t i = (size_t)(hi - 1 - j) * sE + e;
      rb[j] = r[i];
      vb[j] = HASV ? v[i] : 0.f;
    }
  };
  load(t);
  for (; t > 0; t -= kAhead) {
    double rc[kAhead];
    float vc[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) { rc[j] = rb[j]; vc[j] = vb[j]; }
    if (t > kAhead) load(t - kAhead);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kAhead; ++j) step((size_t)(t - 1 - j) * sE + e, rc[j], (double)vc[j]);
  }
}

// Small batches, whose lanes are too few to keep HBM busy or to hide its latency: kEnvs
// environments per workgroup, kSteps steps per chunk. One wave runs the recurrence (a
// lane per environment) over the deltas of chunk c in LDS while the mover threads write out
// chunk c - 1, put the deltas of chunk c + 1 in its place and issue the loads of chunk c + 2.
// Bound by the recurrence's own chain (T = 1000: about 16 cycles a step) once the movers keep
// up: 256 x 1000 without V 17.7 us, against 34 us in the streaming form and 265 us with a memory
// round trip per step.
constexpr int kEnvs = 16, kItems = 8, kMovers = 256, kSteps = kItems * kMovers / kEnvs;
constexpr int kUnroll = 8;
static_assert(kSteps % kUnroll == 0, "whole groups of steps");
template <bool HASV>
__global__ __launch_bounds__(64 + kMovers) void gae_tile_k(int T, int E,
                                                           const double* __restrict__ r,
                                                           const float* __restrict__ v,
                                                           double gamma, double gl,
                                                           double* __restrict__ adv,
                                                           double* __restrict__ ret) {
  // step hi - 1 - q of the chunk that ends at hi in row q of its buffer
  __shared__ double tile[2][kSteps][kEnvs];
  const int nch = (T + kSteps - 1) / kSteps;
  if (threadIdx.x < 64) {   // uniform per wave: the recurrence
    const int el = threadIdx.x % kEnvs;
    double a = 0.0;
    __syncthreads();        // chunk 0's deltas are in place
    for (int c = 0; c < nch; ++c) {
      if (threadIdx.x < kEnvs) {
        double(*tl)[kEnvs] = tile[c & 1];
        // steps past the chunk's end hold zero deltas; their results are not written out
        double d[kUnroll], n[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) n[j] = tl[j][el];
        for (int q = 0; q < kSteps; q += kUnroll) {
#pragma unroll
          for (int j = 0; j < kUnroll; ++j) d[j] = n[j];
          if (q + kUnroll < kSteps) {
#pragma unroll
            for (int j = 0; j < kUnroll; ++j) n[j] = tl[q + kUnroll + j][el];
          }
#pragma unroll
          for (int j = 0; j < kUnroll; ++j) {
            a = d[j] + gl * a;
            tl[q + j][el] = a;
          }
        }
      }
      __syncthreads();
    }
    return;
  }
  const int tid = threadIdx.x - 64, el = tid % kEnvs, row = tid / kEnvs;
  constexpr int kRows = kMovers / kEnvs;
  const int e = blockIdx.x * kEnvs + el;
  const size_t sE = (size_t)E;
  const bool live = e < E;
  double rb[kItems];
  float v0[kItems], v1[kItems], vp[kItems], vc[kItems];   // vp, vc: V_t of chunks c - 1 and c
  auto load = [&](int hi) {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int t = hi - 1 - (row + j * kRows);
      rb[j] = 0.0;
      v0[j] = v1[j] = 0.f;
      if (live && t >= 0) {
        const size_t i = (size_t)t * sE + e;
        rb[j] = r[i];
        if (HASV) {
          v0[j] = v[i];
          v1[j] = v[i + sE];
        }
      }
    }
  };
  auto deltas = [&](double (*tl)[kEnvs]) {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      vp[j] = vc[j];
      vc[j] = v0[j];
      tl[row + j * kRows][el] = (rb[j] + gamma * (double)v1[j]) - (double)v0[j];
    }
  };
  auto write = [&](double (*tl)[kEnvs], int hi) {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int t = hi - 1 - (row + j * kRows);
      if (live && t >= 0) {
        const size_t i = (size_t)t * sE + e;
        const double x = tl[row + j * kRows][el];
        adv[i] = x;
        ret[i] = x + (double)vp[j];
      }
    }
  };
#pragma unroll
  for (int j = 0; j < kItems; ++j) vp[j] = vc[j] = 0.f;
  load(T);
  deltas(tile[0]);
  load(T - kSteps);
  __syncthreads();
  for (int c = 0; c < nch; ++c) {   // the recurrence of chunk c runs beside this
    double(*tl)[kEnvs] = tile[(c + 1) & 1];
    if (c > 0) write(tl, T - (c - 1) * kSteps);
    deltas(tl);
    load(T - (c + 2) * kSteps);
    __syncthreads();
  }
  write(tile[(nch - 1) & 1], T - (nch - 1) * kSteps);
}

}  // namespace

// Up to which batch the tiled form is used: it has a sixteenth of the other's environments per
// wave, so it fills more of the chip, but its rows are read in 16-environment segments. Where
// those start on cache lines (E a multiple of 16; us with V, tiled against streaming, T = 512):
// 4096 environments 17.7 / 31.3, 12288 30.7 / 34.2, 15360 38.0 / 37.0, 65536 213 / 171. Where
// they straddle lines: 5001 23.4 / 34.0, 9999 39.7 / 35.8, 14001 55.0 / 39.2.
constexpr int kTileE = 14336, kTileEOdd = 8192;

hipError_t launch_gae(int T, int E, const double* r, const float* v, double gamma, double lam,
                      double* adv, double* ret, hipStream_t st) {
  const double gl = gamma * lam;
  if (E <= (E % kEnvs ? kTileEOdd : kTileE)) {
    const dim3 grid((E + kEnvs - 1) / kEnvs), block(64 + kMovers);
    if (v) hipLaunchKernelGGL(gae_tile_k<true>, grid, block, 0, st, T, E, r, v, gamma, gl, adv, ret);
    else hipLaunchKernelGGL(gae_tile_k<false>, grid, block, 0, st, T, E, r, v, gamma, gl, adv, ret);
  } else {
    const dim3 grid((E + 63) / 64), block(64);
    if (v) hipLaunchKernelGGL(gae_stream_k<true>, grid, block, 0, st, T, E, r, v, gamma, gl, adv, ret);
    else hipLaunchKernelGGL(gae_stream_k<false>, grid, block, 0, st, T, E, r, v, gamma, gl, adv, ret);
  }
  return hipGetLastError();
}

}  // namespace bsim
