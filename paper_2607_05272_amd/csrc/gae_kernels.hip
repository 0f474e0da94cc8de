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

// One lane per environment, every row access coalesced. Bound by HBM once enough loads are in flight:
// a lane that loads one row, sums it and stores it waits out a memory round trip per step (65536 x
// 1024: 1080 us, 1.7 TB/s), so the rows of the next AHEAD steps are loaded while the current ones are
// summed and stored (8 rows 345 us, 5.45 TB/s; a plain copy reaches 5.2). The more waves there are, the
// fewer rows each needs, and more only scatter the accesses: see launch_gae.
template <bool HASV, int AHEAD, int BLOCK>
__global__ __launch_bounds__(BLOCK) void gae_stream_k(int T, int E, const double* __restrict__ r,
                                                      const float* __restrict__ v, double gamma,
                                                      double gl, double* __restrict__ adv,
                                                      double* __restrict__ ret) {
  const int e = blockIdx.x * BLOCK + threadIdx.x;
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
  for (; t % AHEAD; --t) {
    const size_t i = (size_t)(t - 1) * sE + e;
    step(i, r[i], HASV ? (double)v[i] : 0.0);
  }
  if (t == 0) return;
  double rb[AHEAD];
  float vb[AHEAD];
  auto load = [&](int hi) {
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) {
      const size_t i = (size_t)(hi - 1 - j) * sE + e;
      rb[j] = r[i];
      vb[j] = HASV ? v[i] : 0.f;
    }
  };
  load(t);
  for (; t > 0; t -= AHEAD) {
    double rc[AHEAD];
    float vc[AHEAD];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) { rc[j] = rb[j]; vc[j] = vb[j]; }
    if (t > AHEAD) load(t - AHEAD);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) step((size_t)(t - 1 - j) * sE + e, rc[j], (double)vc[j]);
  }
}

// The largest batches, whose waves alone keep HBM busy: a row at a time, V's load before r's.
__global__ __launch_bounds__(256) void gae_row_k(int T, int E, const double* __restrict__ r,
                                                 const float* __restrict__ v, double gamma, double gl,
                                                 double* __restrict__ adv, double* __restrict__ ret) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= E) return;
  const size_t sE = (size_t)E;
  double a = 0.0, vn = v ? (double)v[(size_t)T * sE + e] : 0.0;
  for (int t = T - 1; t >= 0; --t) {
    const size_t i = (size_t)t * sE + e;
    const double vt = v ? (double)v[i] : 0.0;
    const double delta = (r[i] + gamma * vn) - vt;
    a = delta + gl * a;
    adv[i] = a;
    ret[i] = a + vt;
    vn = vt;
  }
}

// Small batches, whose lanes are too few to keep HBM busy or to hide its latency: kEnvs
// environments per workgroup, kSteps steps per chunk. One wave runs the recurrence (a
// lane per environment) over the deltas of chunk c in LDS while the mover threads write out
// chunk c - 1, put the deltas of chunk c + 1 in its place and issue the loads of chunk c + 2.
// Bound by the recurrence's wave and what feeds it: 256 x 1000 without V 17.1 us, 13.3 of them after
// the launch, about 31 cycles a step, of which the dependent multiplication and addition are 16 (34 us
// in the streaming form, 265 with a memory round trip per step).
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
// 4096 environments 16.9 / 31.2, 12288 30.1 / 34.1, 14336 35.9 / 36.1, 65536 213 / 171. Where
// they straddle lines: 5001 23.4 / 34.0, 9999 39.7 / 35.8, 14001 55.0 / 39.2. Trajectories shorter than
// its chunks of 128 steps leave it little to overlap (with V 14336 x 16 6.6 / 5.3, 14336 x 64 8.6 / 6.2; its
// time over the streaming form's with V at T = 64, 96, 128: 100 environments 1.02, 0.88, 0.76, 4096 1.04,
// 0.88, 0.77, 10000 1.19, 1.02, 0.94; without V at 96, 128, 160: 1.08, 0.96, 0.93, 1.04, 0.96, 0.93 and
// 1.11, 0.95, 0.95).
constexpr int kTileE = 14336, kTileEOdd = 8192;
static bool tiled(int T, int E, bool has_v) {
  return E <= (E % kEnvs ? kTileEOdd : kTileE) && T >= (has_v ? 64 + E / 256 : kSteps);
}
// From which batches on the streaming form loads one row ahead in place of 8, earlier where the waves'
// rows straddle cache lines, and none (us with and without V, 8, 1 and none: 163840 x 300 271 and 241,
// 276 and 267, 456 and 277; 170001 x 300 387 and 341, 306 and 293, 485 and 303; 184320 x 300 318 and 274,
// 293 and 273, 466 and 282; 262144 x 300 427 and 372, 377 and 343, 492 and 339; 393216 x 100 one and none
// 214 and 170, 203 and 169; 524288 x 100 293 and 257, 255 and 254).
constexpr int kAhead1E = 184320, kAhead1EOdd = 163840, kRowE = 393216;

template <bool HASV>
static void launch(int T, int E, const double* r, const float* v, double gamma, double gl,
                   double* adv, double* ret, hipStream_t st) {
  auto go = [&](auto kern, int envs, int block) {
    hipLaunchKernelGGL(kern, dim3((E + envs - 1) / envs), dim3(block), 0, st, T, E, r, v, gamma, gl,
                       adv, ret);
  };
  if (tiled(T, E, HASV)) go(gae_tile_k<HASV>, kEnvs, 64 + kMovers);
  else if (E < (E % kEnvs ? kAhead1EOdd : kAhead1E)) go(gae_stream_k<HASV, 8, 64>, 64, 64);
  else if (E < kRowE) go(gae_stream_k<HASV, 1, 256>, 256, 256);
  else go(gae_row_k, 256, 256);
}

hipError_t launch_gae(int T, int E, const double* r, const float* v, double gamma, double lam,
                      double* adv, double* ret, hipStream_t st) {
  if (v) launch<true>(T, E, r, v, gamma, gamma * lam, adv, ret, st);
  else launch<false>(T, E, r, v, gamma, gamma * lam, adv, ret, st);
  return hipGetLastError();
}

}  // namespace bsim
