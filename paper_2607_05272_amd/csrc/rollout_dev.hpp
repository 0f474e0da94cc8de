// rollout_dev.hpp -- the fused rollout: one launch runs every tick of a rollout, the policy
// (paper Sec. 4.2) and the learned system's tick (Sec. 3.1, Sec. 4.1) alternating inside each
// workgroup.
//
// With a few thousand environments the per-tick kernels are bound by latency, not by work: a
// launch's start, its first loads of the state and its drain cost more than its arithmetic,
// twice per tick. Environments never interact, so a workgroup can own a tile of them for the
// whole rollout and keep what a tick needs on the CU: the environments' state in LDS (and their
// request rings, where they fit), every wave's share of the policy's weights in registers,
// the observation and the actions passed between the two phases in LDS. Only the trajectory
// is written to memory, and the state at the end; nothing is ever exchanged between
// workgroups, so they run without any grid-wide synchronisation (a grid larger than the chip
// holds simply runs in rounds).
//
// Bound by the chain of one wave's instructions through a tick, at one or two waves per SIMD (us
// per tick, state and weights through L2 before and as here): the 8-64-64-6 network 10.2 -> 5.1
// at 256 environments (of 12500 cycles 3300 in the policy's layers, 1700 in the sampler, 2500
// in loads and events, 2500 at the end of the tick, the rest at barriers), the 12-128-128-6 one
// 8.4 -> 6.5 at 4096, the 32-256-256-24 one 18.6 -> 7.7 at 2000 and 19.8 -> 14.1 at 16384, the
// 64-256-256-48 one 40.6 -> 13.7 at 1024 and 36.0 -> 26.9 at 16384.
//
// The tick is the per-tick kernel's own device code (sim_dev.hpp), and every policy sum takes
// the per-tick kernels' operands in their order (policy_dev.hpp), so every output is
// bit-identical to the per-tick launches'.
#pragma once
#include "policy_dev.hpp"
#include "sim_dev.hpp"

namespace bsim {
namespace {

// ---- the policy on a workgroup's rows, weights in registers --------------------------------
// fp32 policies: 16 rows, four waves (see layer() in policy_dev.hpp: activations the A operand,
// a quarter of the output columns per wave, the bias added after the sum).
template <int FP, int H1, int H2, int AP>
struct NetF32 {
  static constexpr int NW = 4, ROWS = 16, KM = AP / 6, kAP = AP;
  static constexpr bool kBf16 = false;
  static constexpr int T1 = H1 / 16 / NW, T2 = H2 / 16 / NW;
  static_assert(H1 % (16 * NW) == 0 && H2 % (16 * NW) == 0 && AP == 16, "tiles");
  static constexpr int SX = FP + 4, S1 = H1 + 4, S2 = H2 + 4, SL = AP + 1;
  static constexpr size_t X_BYTES = (size_t)ROWS * SX * 4;
  static constexpr size_t LDS = X_BYTES + (size_t)ROWS * (S1 + S2 + SL) * 4;
  float w1[T1][FP / 4], w2[T2][H1 / 4], w3[H2 / 4], b1[T1], b2[T2], b3;

  __device__ __forceinline__ void load(const MlpParams& m, unsigned char*) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kq = lane >> 4;
    const float* W1 = static_cast<const float*>(m.w1);
    const float* W2 = static_cast<const float*>(m.w2);
    const float* W3 = static_cast<const float*>(m.w3);
#pragma unroll
    for (int c = 0; c < T1; ++c) {
      const int col = (wave + 4 * c) * 16 + r16;
      b1[c] = m.b1[col];
#pragma unroll
      for (int ks = 0; ks < FP / 4; ++ks) w1[c][ks] = W1[(size_t)col * FP + ks * 4 + kq];
    }
#pragma unroll
    for (int c = 0; c < T2; ++c) {
      const int col = (wave + 4 * c) * 16 + r16;
      b2[c] = m.b2[col];
#pragma unroll
      for (int ks = 0; ks < H1 / 4; ++ks) w2[c][ks] = W2[(size_t)col * H1 + ks * 4 + kq];
    }
    b3 = m.b3[r16];
#pragma unroll
    for (int ks = 0; ks < H2 / 4; ++ks) w3[ks] = W3[(size_t)r16 * H2 + ks * 4 + kq];
  }

  template <int K, int T, bool LAST>
  __device__ __forceinline__ static void layer_reg(const float* in, int sin, const float (&w)[T][K / 4],
                                                   const float (&b)[T], float* out, int sout) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kq = lane >> 4;
    f32x4 acc[T];
#pragma unroll
    for (int c = 0; c < T; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float a[K / 4];
#pragma unroll
    for (int ks = 0; ks < K / 4; ++ks) a[ks] = in[r16 * sin + ks * 4 + kq];
#pragma unroll
    for (int ks = 0; ks < K / 4; ++ks)
#pragma unroll
      for (int c = 0; c < T; ++c) acc[c] = F32Mode::mfma(a[ks], w[c][ks], acc[c]);
#pragma unroll
    for (int c = 0; c < T; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = acc[c][i] + b[c];
        out[(kq * 4 + i) * sout + (LAST ? 0 : (wave + 4 * c) * 16) + r16] = LAST ? v : gelu(v);
      }
  }

  // logits (and value) of the rows in x into the returned buffer [row][SL]; us: each row's
  // ACTION uniform, drawn by a wave that has no part in the output layer
  template <class Draw>
  __device__ __forceinline__ float* forward(unsigned char* smem, Draw&& draw) {
    float* xs = reinterpret_cast<float*>(smem);
    float* h1 = xs + ROWS * SX;
    float* h2 = h1 + ROWS * S1;
    float* lg = h2 + ROWS * S2;
    layer_reg<FP, T1, false>(xs, SX, w1, b1, h1, S1);
    __syncthreads();
    layer_reg<H1, T2, false>(h1, S1, w2, b2, h2, S2);
    __syncthreads();
    if (threadIdx.x < 64) {
      const float(&w)[1][H2 / 4] = reinterpret_cast<const float(&)[1][H2 / 4]>(w3);
      const float b[1] = {b3};
      layer_reg<H2, 1, true>(h2, S2, w, b, lg, SL);
    } else if (threadIdx.x < 128) {
      draw((int)threadIdx.x - 64);
    }
    return lg;
  }
  // feature pair i, i + 1 (i even) of a row
  __device__ __forceinline__ static void put(unsigned char* smem, int row, int i, float a, float b) {
    float* xs = reinterpret_cast<float*>(smem) + row * SX + i;
    xs[0] = a;
    xs[1] = b;
  }
};

// bf16 policies: 16 RT rows, NW waves (see policy_tile_bf16 in policy_dev.hpp: weights the A
// operand in fragment order, the bias the accumulators' first value, GELU and the rounding to
// bf16 in the epilogue).
template <int FP, int H1, int H2, int AP, int RT, int NWAVES>
struct NetBf16 {
  static constexpr int NW = NWAVES, ROWS = 16 * RT, KM = AP / 6, kAP = AP;
  static constexpr bool kBf16 = true;
  static constexpr int T1 = H1 / 16 / NW, T2 = H2 / 16 / NW, NT = AP / 16;
  static_assert(H1 % (16 * NW) == 0 && H2 % (16 * NW) == 0, "whole tiles per wave");
  // the output layer's NT x RT tiles over the waves, RTN row tiles of one column tile each
  static constexpr int RTN = NT * RT > NW ? NT * RT / NW : 1;
  static_assert(RT % RTN == 0, "row-tile runs of the output layer");
  static constexpr int K1 = FP / 32, K2 = H1 / 32, K3 = H2 / 32;
  static constexpr int SX = FP + 8, S1 = H1 + 8, S2 = H2 + 8, SL = AP + 4;
  static constexpr size_t X_BYTES = (size_t)ROWS * SX * 2;
  static constexpr size_t H1_BYTES = (size_t)ROWS * S1 * 2, L_BYTES = (size_t)ROWS * SL * 4;
  static constexpr size_t Q_BYTES = H1_BYTES > L_BYTES ? H1_BYTES : L_BYTES;   // h1, then logits
  static constexpr size_t LDS = X_BYTES + Q_BYTES + (size_t)ROWS * S2 * 2 + (size_t)(H1 + H2 + AP) * 4;
  bf16x8 w1[T1][K1], w2[T2][K2], w3[K3];

  __device__ __forceinline__ static int wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
  __device__ __forceinline__ static float* biases(unsigned char* smem) {
    return reinterpret_cast<float*>(smem + X_BYTES + Q_BYTES + (size_t)ROWS * S2 * 2);
  }
  __device__ __forceinline__ static bool out_wave() { return wave() < NT * RT / RTN; }

  __device__ __forceinline__ void load(const MlpParams& m, unsigned char* smem) {
    const int lane = threadIdx.x & 63, wv = wave();
    auto frag = [&](const void* W, int KS, int tile, int ks) {
      return *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(W) +
                                              ((size_t)tile * KS + ks) * 512 + lane * 8);
    };
#pragma unroll
    for (int c = 0; c < T1; ++c)
#pragma unroll
      for (int ks = 0; ks < K1; ++ks) w1[c][ks] = frag(m.w1, K1, wv + NW * c, ks);
#pragma unroll
    for (int c = 0; c < T2; ++c)
#pragma unroll
      for (int ks = 0; ks < K2; ++ks) w2[c][ks] = frag(m.w2, K2, wv + NW * c, ks);
#pragma unroll
    for (int ks = 0; ks < K3; ++ks) w3[ks] = frag(m.w3, K3, wv % NT, ks);
    float* b = biases(smem);
    for (int q = threadIdx.x; q < H1 + H2 + AP; q += NW * 64)
      b[q] = q < H1 ? m.b1[q] : q < H1 + H2 ? m.b2[q - H1] : m.b3[q - H1 - H2];
  }

  template <int K, int T, int R>
  __device__ __forceinline__ static void mma(const uint16_t* act, int sa, const bf16x8 (&w)[T][K],
                                             const float* bias, int tile0, int rt0,
                                             f32x4 (&acc)[T][R]) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int c = 0; c < T; ++c) {
      const f32x4 bv = *reinterpret_cast<const f32x4*>(bias + (tile0 + NW * c) * 16 + kq * 4);
#pragma unroll
      for (int rt = 0; rt < R; ++rt) acc[c][rt] = bv;
    }
    const uint16_t* a = act + (rt0 * 16 + r16) * sa + kq * 8;
#pragma unroll
    for (int ks = 0; ks < K; ++ks)
#pragma unroll
      for (int rt = 0; rt < R; ++rt) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(a + rt * 16 * sa + ks * 32);
#pragma unroll
        for (int c = 0; c < T; ++c)
          acc[c][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[c][ks], b, acc[c][rt], 0, 0, 0);
      }
  }
  template <int T>
  __device__ __forceinline__ static void hidden(const f32x4 (&acc)[T][RT], uint16_t* out, int so) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int c = 0; c < T; ++c)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        *reinterpret_cast<u32x2*>(out + (rt * 16 + r16) * so + (wave() + NW * c) * 16 + kq * 4) =
            gelu_pack4(acc[c][rt]);
  }

  template <class Draw>
  __device__ __forceinline__ float* forward(unsigned char* smem, Draw&& draw) {
    uint16_t* xs = reinterpret_cast<uint16_t*>(smem);
    uint16_t* h1 = reinterpret_cast<uint16_t*>(smem + X_BYTES);
    uint16_t* h2 = reinterpret_cast<uint16_t*>(smem + X_BYTES + Q_BYTES);
    float* lg = reinterpret_cast<float*>(smem + X_BYTES);
    const float* b = biases(smem);
    {
      f32x4 acc[T1][RT];
      mma<K1, T1, RT>(xs, SX, w1, b, wave(), 0, acc);
      hidden<T1>(acc, h1, S1);
    }
    __syncthreads();
    {
      f32x4 acc[T2][RT];
      mma<K2, T2, RT>(h1, S1, w2, b + H1, wave(), 0, acc);
      draw((int)threadIdx.x);
      hidden<T2>(acc, h2, S2);
    }
    __syncthreads();
    if (out_wave()) {
      const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
      const int tile = wave() % NT, rt0 = (wave() / NT) * RTN;
      f32x4 acc[1][RTN];
      const bf16x8(&w)[1][K3] = reinterpret_cast<const bf16x8(&)[1][K3]>(w3);
      mma<K3, 1, RTN>(h2, S2, w, b + H1 + H2, tile, rt0, acc);
#pragma unroll
      for (int rt = 0; rt < RTN; ++rt)
        *reinterpret_cast<f32x4*>(lg + ((rt0 + rt) * 16 + r16) * SL + tile * 16 + kq * 4) = acc[0][rt];
    }
    return lg;
  }
  __device__ __forceinline__ static void put(unsigned char* smem, int row, int i, float a, float b) {
    reinterpret_cast<uint32_t*>(smem)[(row * SX + i) >> 1] = pack_bf16_pair(a, b);
  }
};

// The same with the weights read from L2 every tick, two tiles at a time and two steps ahead, for
// networks whose share per wave would take the registers that the tick needs.
template <int FP, int H1, int H2, int AP, int RT, int NWAVES>
struct NetBf16Stream : NetBf16<FP, H1, H2, AP, RT, NWAVES> {
  typedef NetBf16<FP, H1, H2, AP, RT, NWAVES> B;
  using B::NW; using B::NT; using B::RTN;
  MlpParams m;
  __device__ __forceinline__ void load(const MlpParams& p, unsigned char* smem) {
    m = p;
    float* b = B::biases(smem);
    for (int q = threadIdx.x; q < H1 + H2 + AP; q += NW * 64)
      b[q] = q < H1 ? m.b1[q] : q < H1 + H2 ? m.b2[q - H1] : m.b3[q - H1 - H2];
  }
  template <int K, int T, int R>
  __device__ __forceinline__ static void mma_stream(const uint16_t* act, int sa, const void* W,
                                                    const float* bias, int tile0, int rt0,
                                                    f32x4 (&acc)[T][R]) {
    constexpr int D = K < 2 ? K : 2, S = D + 1;
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
    const uint16_t* wp[T];
    bf16x8 w[S][T], b[2][R];
#pragma unroll
    for (int c = 0; c < T; ++c) {
      wp[c] = static_cast<const uint16_t*>(W) + (size_t)(tile0 + NW * c) * K * 512 + lane * 8;
#pragma unroll
      for (int s = 0; s < D; ++s) w[s][c] = *reinterpret_cast<const bf16x8*>(wp[c] + s * 512);
      const f32x4 bv = *reinterpret_cast<const f32x4*>(bias + (tile0 + NW * c) * 16 + kq * 4);
#pragma unroll
      for (int rt = 0; rt < R; ++rt) acc[c][rt] = bv;
    }
    const uint16_t* a = act + (rt0 * 16 + r16) * sa + kq * 8;
#pragma unroll
    for (int rt = 0; rt < R; ++rt) b[0][rt] = *reinterpret_cast<const bf16x8*>(a + rt * 16 * sa);
#pragma unroll
    for (int ks = 0; ks < K; ++ks) {
      if (ks + 1 < K) {
#pragma unroll
        for (int rt = 0; rt < R; ++rt)
          b[(ks + 1) & 1][rt] = *reinterpret_cast<const bf16x8*>(a + rt * 16 * sa + (ks + 1) * 32);
      }
      if (ks + D < K) {
#pragma unroll
        for (int c = 0; c < T; ++c)
          w[(ks + D) % S][c] = *reinterpret_cast<const bf16x8*>(wp[c] + (ks + D) * 512);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int rt = 0; rt < R; ++rt)
#pragma unroll
        for (int c = 0; c < T; ++c)
          acc[c][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks % S][c], b[ks & 1][rt],
                                                               acc[c][rt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  template <int K, int T>
  __device__ __forceinline__ static void layer_stream(const uint16_t* in, int si, const void* W,
                                                      const float* bias, uint16_t* out, int so) {
    constexpr int P = T < 2 ? T : 2;
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int c0 = 0; c0 < T; c0 += P) {
      f32x4 acc[P][RT];
      const int tile0 = B::wave() + NW * c0;
      mma_stream<K, P, RT>(in, si, W, bias, tile0, 0, acc);
#pragma unroll
      for (int c = 0; c < P; ++c)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          *reinterpret_cast<u32x2*>(out + (rt * 16 + r16) * so + (tile0 + NW * c) * 16 + kq * 4) =
              gelu_pack4(acc[c][rt]);
    }
  }
  template <class Draw>
  __device__ __forceinline__ float* forward(unsigned char* smem, Draw&& draw) {
    uint16_t* xs = reinterpret_cast<uint16_t*>(smem);
    uint16_t* h1 = reinterpret_cast<uint16_t*>(smem + B::X_BYTES);
    uint16_t* h2 = reinterpret_cast<uint16_t*>(smem + B::X_BYTES + B::Q_BYTES);
    float* lg = reinterpret_cast<float*>(smem + B::X_BYTES);
    const float* b = B::biases(smem);
    layer_stream<FP / 32, H1 / 16 / NW>(xs, B::SX, m.w1, b, h1, B::S1);
    __syncthreads();
    layer_stream<H1 / 32, H2 / 16 / NW>(h1, B::S1, m.w2, b + H1, h2, B::S2);
    draw((int)threadIdx.x);
    __syncthreads();
    if (B::out_wave()) {
      const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
      const int tile = B::wave() % NT, rt0 = (B::wave() / NT) * RTN;
      f32x4 acc[1][RTN];
      mma_stream<H2 / 32, 1, RTN>(h2, B::S2, m.w3, b + H1 + H2, tile, rt0, acc);
#pragma unroll
      for (int rt = 0; rt < RTN; ++rt)
        *reinterpret_cast<f32x4*>(lg + ((rt0 + rt) * 16 + r16) * B::SL + tile * 16 + kq * 4) =
            acc[0][rt];
    }
    return lg;
  }
};

// ---- the workgroup's environments in LDS -----------------------------------------------------
// State arrays [field][ROWS] (K servers up to KM, classes up to CM), then the rate averages.
template <int CM, int KM, int ROWS>
struct TileState {
  double hts[CM][ROWS], busy[KM][ROWS], sums[2][ROWS], next_sw[ROWS], next_arr[ROWS];
  uint64_t chk[ROWS];
  double ewma[4][ROWS];
  uint32_t qpack[ROWS], hpack[ROWS], meta[KM][ROWS], cnt[kNcnt][ROWS], proc[ROWS], tr_idx[ROWS];
  // of the tick at hand: the head-of-line request's time, weighted latencies, requests
  // dispatched and arrivals
  double hts_h[ROWS], Lw[ROWS];
  int n_k[ROWS], A_k[ROWS];

  __device__ __forceinline__ SysState view() {
    SysState s{};
    s.qpack = qpack; s.hpack = hpack; s.hts = &hts[0][0]; s.busy = &busy[0][0];
    s.meta = &meta[0][0]; s.cnt = &cnt[0][0]; s.sums = &sums[0][0]; s.chk = chk;
    s.proc = proc; s.next_sw = next_sw; s.next_arr = next_arr; s.tr_idx = tr_idx;
    return s;
  }
  // every field of rows 0 .. n - 1 through f(LDS element, memory element); memory rows of length
  // p.E from environment e0
  template <class F>
  __device__ __forceinline__ void each(const SimParams& p, const EnvState& g, int e0, int n, F&& f) {
    const SysState& G = g.sys[0];
    const size_t E = (size_t)p.E;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const size_t e = (size_t)e0 + i;
      f(qpack[i], G.qpack[e]);
      f(hpack[i], G.hpack[e]);
      f(chk[i], G.chk[e]);
      f(proc[i], G.proc[e]);
      f(next_sw[i], G.next_sw[e]);
      f(next_arr[i], G.next_arr[e]);
      f(tr_idx[i], G.tr_idx[e]);
#pragma unroll
      for (int c = 0; c < CM; ++c)
        if (c < p.C) f(hts[c][i], G.hts[c * E + e]);
#pragma unroll
      for (int c = 0; c < kNcnt; ++c) f(cnt[c][i], G.cnt[c * E + e]);
      f(sums[0][i], G.sums[e]);
      f(sums[1][i], G.sums[E + e]);
#pragma unroll
      for (int c = 0; c < 4; ++c) f(ewma[c][i], g.ewma[c * E + e]);
      for (int j = 0; j < p.K; ++j) {
        f(busy[j][i], G.busy[j * E + e]);
        f(meta[j][i], G.meta[j * E + e]);
      }
    }
  }
};

// The tick's checksum and reward of row r (environment e) with `done` more requests completed.
template <int CM, class State>
__device__ __forceinline__ void close_row(const SimParams& p, State& S, int r, int e, uint32_t qp,
                                          int A_k, uint32_t done, double* rew, uint64_t* rchk) {
  Count C;
  C.chk = S.chk[r];
  C.n_k = S.n_k[r];
  C.Lw = S.Lw[r];
  C.c[C_DONE] = S.cnt[C_DONE][r] + done;
  C.c[C_DROP] = S.cnt[C_DROP][r];
  Queue<CM> Q;
  Q.qp = qp;
  const double rw = close_tick(Q, C, p, S.proc[r], A_k);
  S.chk[r] = C.chk;
  S.cnt[C_DONE][r] = C.c[C_DONE];
  if (rew) rew[e] = rw;
  if (rchk) rchk[e] = C.chk;
}

// One tick of the wave's rows r0 .. r0 + lpw - 1 (environments e0 + r0 .., `n` of the workgroup's
// rows live), state in LDS. The first lpw lanes take the events, one row each; then the end of
// the tick (completions, checksum, reward, rate averages, observation), which is a chain of
// short dependent steps in one lane (3000 to 8000 of a tick's cycles for 1 to 8 servers), is
// shared by eight lanes per row: every eighth server, a class or the queues' total, a rate each.
// DEFER: the checksum and the reward, which the next tick's policy does not need, are left to the
// caller (close_row).
template <class Net, int CM, bool INL, int LN, bool DEFER, class State>
__device__ __forceinline__ void tile_tick(const SimParams& p, State& S, uint32_t* err,
                                          double* rings, uint64_t seed, uint32_t k, int e0, int r0,
                                          int lpw, int n, Stage<kStageLearned, LN>& st,
                                          uint32_t staged, const uint8_t* act,
                                          unsigned char* smem, const ObsPairs& out, double* rew,
                                          uint64_t* rchk) {
  constexpr int ROWS = Net::ROWS;
  static_assert(LN <= 8, "eight lanes per row");
  const SysState G = S.view();
  const int lane = threadIdx.x & 63;
  {
    const bool live = lane < lpw && r0 + lane < n;
    const int r = live ? r0 + lane : 0;
    auto load = [&](Queue<CM>& Q, Count& C, Arrivals& A, int& sv, int& b, double& busy_s,
                    uint32_t& meta_s) {
      const int a = live ? act[r] : 0;   // sampled here: always a valid action
      load_queue(Q, G, p, ROWS, r);
      Q.ring = rings + (size_t)r * p.C * p.N;
      load_count(C, G, ROWS, r);
      load_arrivals(A, G, p, r, e0 + r);
      sv = a / 6;
      b = 1 << (a % 6);
      busy_s = G.busy[sv * ROWS + r];
      meta_s = G.meta[sv * ROWS + r];
    };
    auto store = [&](Queue<CM>& Q, Count& C, Arrivals& A, int sv, int b, double busy_s,
                     uint32_t meta_s, bool dirty_s, int A_k) {
      if (!live) return;
      store_queue(Q, G, p, ROWS, r);
      store_count(C, G, ROWS, r);
      store_arrivals(A, G, p, r);
      if (dirty_s) {
        G.busy[sv * ROWS + r] = busy_s;
        G.meta[sv * ROWS + r] = meta_s;
      }
      S.hts_h[r] = Q.hts_h;
      S.Lw[r] = C.Lw;
      S.n_k[r] = C.n_k;
      S.A_k[r] = A_k;
    };
    tick_events<CM, INL, LN>(p, err, seed, k, e0 + r0, live, e0 + r, st, staged, load, store);
  }
  wave_sync_lds();
  const int g8 = lane >> 3, s = lane & 7, r = r0 + g8;
  const bool live = g8 < lpw && r < n;
  if (!live) return;   // whole groups of eight lanes
  const double t1 = (double)(k + 1) * p.dt;
  ObsPairs ob = out;
  ob.e = e0 + r;
  auto put = [&](int i, double v0, double v1) {
    Net::put(smem, r, i, (float)v0, (float)v1);
    if (ob.cur || ob.traj) ob.put(i, v0, v1);
  };
  // servers s, s + 8, ...: completions before t1 and their features
  const int per = p.K > 1 ? 4 : 2;
  int done = 0;
  for (int j = s; j < p.K; j += 8) {
    const double bu = S.busy[j][r];
    uint32_t m = S.meta[j][r];
    const uint32_t infl = m & 0xffu;
    if (infl > 0 && bu < t1) {
      done += (int)infl;
      m &= ~0xffu;
      S.meta[j][r] = m;
    }
    const int base = 2 + per * j;
    put(base, bu > t1 ? 1.0 : 0.0, (double)((m >> 8) & 0xffu) * 0.03125);
    if (p.K > 1) {
      const uint32_t lc = (m >> 16) & 0xffu;
      put(base + 2, (bu > t1 ? bu - t1 : 0.0) * p.inv_tw,
          (double)((lc == 0xffu ? -1 : (int)lc) + 1) * p.inv_c);
    }
  }
  done += dpp8<kDppXor1>(done);
  done += dpp8<kDppXor2>(done);
  done += dpp8<kDppHalfMirror>(done);
  const uint32_t qp = S.qpack[r];
  const int qsum = (int)((qp & 0xffu) + ((qp >> 8) & 0xffu) + ((qp >> 16) & 0xffu) + (qp >> 24));
  const int A_k = S.A_k[r];
  int i = 2 + per * p.K;
  // class s's queue, or (s = C) all of them
  if (s <= p.C && (s == p.C || p.C > 1)) {
    const int q = s < p.C ? (int)((qp >> (8 * s)) & 0xffu) : qsum;
    const double ts = s < p.C ? S.hts[s < CM ? s : 0][r] : S.hts_h[r];
    put(s < p.C ? i + 2 * s : 0, (double)q * p.inv_n, (q > 0 ? t1 - ts : 0.0) * p.inv_tw);
  }
  if (p.C > 1) i += 2 * p.C;
  // rate average s, features in pairs
  {
    double ew = S.ewma[s & 3][r];
    const double w = s == 0 ? 1.0 : s == 1 ? 0.25 : s == 2 ? 0.0625 : 0.015625;
    ew = ew + w * ((double)A_k - ew);
    const double v = ew * p.inv_rs;
    const double v1 = __hiloint2double(dpp8<kDppXor1>(__double2hiint(v)),
                                       dpp8<kDppXor1>(__double2loint(v)));
    if (s < 4) S.ewma[s][r] = ew;
    if (s == 0 || s == 2) put(i + s, v, v1);
  }
  if (ob.traj)   // features past the state's: zero (the policy's rows hold zeros there)
    for (int f = i + 4 + s; f < p.F; f += 8) ob.traj[(size_t)f * ob.E + ob.e] = 0.0f;
  if (s == 7) {
    if constexpr (DEFER) S.cnt[C_DONE][r] += (uint32_t)done;
    else close_row<CM>(p, S, r, ob.e, qp, A_k, (uint32_t)done, rew, rchk);
  }
}

// T ticks from k0 for environments e0 = blockIdx.x * rows .. (rows <= ROWS, a multiple of the
// waves). Trajectory rows as in the per-tick rollout: act, logp, value, rew and rchk [T][E], obs
// [T + 1][F][E] from row 1 (row 0, the observation before the first tick, is not written here),
// value row T for the observation after the last tick. RL: the rings in LDS, else in memory.
template <class Net, int CM, bool RL>
__global__ __launch_bounds__(Net::NW * 64) __attribute__((amdgpu_waves_per_eu(2))) void rollout_fused_k(
    SimParams p, EnvState g, MlpParams m, uint32_t k0, int T, int rows, RolloutOut o) {
  constexpr int ROWS = Net::ROWS, NW = Net::NW, NTHR = NW * 64, LN = ROWS / NW;
  // the fp64 elementary functions inline with three or four classes (as in the per-tick kernels;
  // 8 servers 28.6 us per tick against 29.4 called, with fewer classes even)
  constexpr bool kInl = CM >= 4;
  typedef TileState<CM, Net::KM, ROWS> State;
  __shared__ Stage<kStageLearned, LN> stage[NW];
  __shared__ State state;
  __shared__ float us[ROWS];
  __shared__ uint8_t act[ROWS];
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  double* ring_lds = reinterpret_cast<double*>(smem + Net::LDS);
  const uint64_t seed = *g.seed;   // the episode seed, written by reset_k
  const int e0 = blockIdx.x * rows, tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lpw = rows / NW;
  const int n = min(rows, p.E - e0);
  const size_t E = (size_t)p.E, F = (size_t)p.F;
  double* ring_mem = g.sys[0].ring + (size_t)e0 * p.C * p.N;
  const int nring = n * p.C * p.N;

  Net net;
  net.load(m, smem);
  for (int q = tid; q < (int)(Net::X_BYTES / 4); q += NTHR) reinterpret_cast<uint32_t*>(smem)[q] = 0u;
  state.each(p, g, e0, n, [](auto& l, auto& v) { l = v; });
  if constexpr (RL)
    for (int q = tid; q < nring; q += NTHR) ring_lds[q] = ring_mem[q];
  __syncthreads();
  for (int q = tid; q < n * ((p.F + 1) / 2); q += NTHR) {
    const int r = q % n, i = 2 * (q / n);
    Net::put(smem, r, i, g.obs[(size_t)i * E + e0 + r],
             i + 1 < p.F ? g.obs[(size_t)(i + 1) * E + e0 + r] : 0.f);
  }
  __syncthreads();
  // the tick's first ARRIVAL blocks: with fewer rows than eight per wave, staged by the waves that
  // have no rows to sample, else by each wave for its own rows (one block per lane)
  constexpr int kIdle = NW - ROWS / 8;
  const int npre = p.arrival_kind == 1 ? 0 : kIdle > 0 ? 8 : 64 / LN;
  // the last of those waves also takes the previous tick's checksums and rewards, off the chain of
  // the tick (us per tick, 256 environments of one server 5.40 -> 5.10, 128 of the 12-128-128-6 network
  // 6.55 -> 6.09; with four classes it costs registers, 8192 with 8 servers 22.2 -> 23.0)
  constexpr bool kDefer = kIdle > 0 && CM <= 2;

  auto close = [&](int i) {   // tick i's, a row per lane
    const int r = tid & 63;
    const size_t row = (size_t)i * E;
    if (r < n)
      close_row<CM>(p, state, r, e0 + r, state.qpack[r], state.A_k[r], 0u,
                    o.rew ? o.rew + row : nullptr, o.rchk ? o.rchk + row : nullptr);
  };

  for (int i = 0; i <= T; ++i) {
    const uint32_t k = k0 + (uint32_t)i;
    const size_t row = (size_t)i * E;
    if (i == T && !o.value) break;
    const float* lg = net.forward(smem, [&](int r) {
      if (r < ROWS) us[r] = action_uniform(seed, (uint32_t)(r < n ? e0 + r : 0), k);
    });
    __syncthreads();
    const bool last = i == T;   // only the value of the observation after the last tick
    sample_rows<Net::kAP, ROWS, NTHR>(lg, Net::SL, m, e0, seed, k, last ? nullptr : o.act + row,
                                      !last && o.logp ? o.logp + row : nullptr,
                                      o.value ? o.value + row : nullptr, nullptr, us, n, act);
    if (last) break;
    if constexpr (kDefer) {
      if (wave == NW - 1 && i > 0) close(i - 1);
    }
    if constexpr (kIdle > 0) {
      const int w0 = wave - ROWS / 8;
      if (w0 >= 0)
        for (int q = w0 * 64 + (tid & 63); q < n * npre; q += kIdle * 64) {
          const int r = q / npre;
          stage_block<CM, kStageLearned, true, LN>(stage[r / lpw], p, seed, (uint32_t)(e0 + r), k,
                                                   (uint32_t)(q % npre), r % lpw);
        }
    }
    __syncthreads();   // the tile's actions are written
    const int r0 = wave * lpw;
    if constexpr (kIdle <= 0) {
      const int q = tid & 63;
      if (npre > 0 && q / npre < lpw && r0 + q / npre < n)
        stage_block<CM, kStageLearned, true, LN>(stage[wave], p, seed,
                                                 (uint32_t)(e0 + r0 + q / npre), k,
                                                 (uint32_t)(q % npre), q / npre);
      wave_sync_lds();
    }
    const bool end = i + 1 == T;
    const ObsPairs out{end ? g.obs : nullptr, o.obs ? o.obs + (size_t)(i + 1) * F * E : nullptr,
                       Net::kBf16 && end ? g.obs_bf : nullptr, E, 0};
    tile_tick<Net, CM, kInl, LN, kDefer>(p, state, g.err, RL ? ring_lds : ring_mem, seed, k, e0, r0, lpw, n,
                                 stage[wave], (uint32_t)npre, act, smem, out,
                                 o.rew ? o.rew + row : nullptr, o.rchk ? o.rchk + row : nullptr);
    __syncthreads();   // the tile's next observation and state are written
  }
  if constexpr (kDefer) {
    if (wave == NW - 1) close(T - 1);
    __syncthreads();
  }
  state.each(p, g, e0, n, [](auto& l, auto& v) { v = l; });
  if constexpr (RL)
    for (int q = tid; q < nring; q += NTHR) ring_mem[q] = ring_lds[q];
}

// ---- host ------------------------------------------------------------------------------------
template <class Net, int CM, bool RL>
struct Fused {
  static constexpr auto kern = rollout_fused_k<Net, CM, RL>;
  static size_t dynamic_lds(const SimParams& p) {
    return Net::LDS + (RL ? (size_t)Net::ROWS * p.C * p.N * 8 : 0);
  }
  static constexpr size_t kStatic =
      sizeof(Stage<kStageLearned, Net::ROWS / Net::NW>) * Net::NW +
      sizeof(TileState<CM, Net::KM, Net::ROWS>) + Net::ROWS * 5 + 64;
  // (the rings' size is the context's, the limit the kernel's: the most that fits)
  static hipError_t allow() {
    static std::atomic<uint64_t> lds_on{0};
    return allow_lds((const void*)kern, kLdsMax - kStatic, lds_on);
  }
  static bool fits(const SimParams& p) { return kStatic + dynamic_lds(p) <= kLdsMax; }
  // environments resident at once
  static hipError_t capacity(const SimParams& p, int cus, int* envs) {
    hipError_t e = allow();
    int per_cu = 0;
    if (e == hipSuccess)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, Net::NW * 64, dynamic_lds(p));
    *envs = per_cu * cus * Net::ROWS;
    return e;
  }
  static hipError_t launch(const SimParams& p, const EnvState& s, const MlpParams& m, uint32_t k0,
                           int T, const RolloutOut& o, int cap, hipStream_t st) {
    // a batch smaller than the chip takes is spread over more workgroups of fewer rows each: a
    // wave's tick lasts as long as its busiest environment
    int rows = Net::ROWS;
    if (p.E < cap) {
      const int slots = cap / Net::ROWS;
      rows = (p.E + slots - 1) / slots;
      rows = (rows + Net::NW - 1) / Net::NW * Net::NW;
    }
    const hipError_t e = allow();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((p.E + rows - 1) / rows), dim3(Net::NW * 64), dynamic_lds(p), st,
                       p, s, m, k0, T, rows, o);
    return hipGetLastError();
  }
};

// The form for a batch among `with`'s (with(f) calls f(number, Fused<...>{}) on each, in growing
// order of what they hold): the first that holds the whole batch at once, else the largest.
template <class With>
hipError_t pick_form(const SimParams& p, FusedPlan* plan, With&& with) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  plan->cap = 0;
  with([&](int id, auto f) {
    if (e != hipSuccess || plan->cap >= p.E || !f.fits(p)) return;
    int cap = 0;
    e = f.capacity(p, cus, &cap);
    if (e == hipSuccess && cap > plan->cap) *plan = FusedPlan{id, cap};
  });
  return e;
}
template <class With>
hipError_t launch_form(const SimParams& p, const EnvState& s, const MlpParams& m,
                       const FusedPlan& plan, uint32_t k0, int T, const RolloutOut& o,
                       hipStream_t st, With&& with) {
  hipError_t e = hipErrorNotSupported;
  with([&](int id, auto f) {
    if (id == plan.form) e = f.launch(p, s, m, k0, T, o, plan.cap, st);
  });
  return e;
}

}  // namespace
}  // namespace bsim
