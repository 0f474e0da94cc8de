// mlp_kernels.hip -- the policy MLP kernels (paper Sec. 4.2), fused with action sampling:
// policy_k (fp32 policies) and policy_bf16_k (bf16 policies), each one workgroup's share of
// the batch as described in policy_dev.hpp, plus the weight repacking and initialisation.
#include <type_traits>

#include "policy_dev.hpp"

namespace bsim {
namespace {

template <class M, int FP, int H1, int H2, int AP, int RT, bool DBG>
__global__ __launch_bounds__(kThreads) void policy_k(MlpParams m, int b0, const float* __restrict__ obs,
                                                     const uint64_t* __restrict__ seedp, uint32_t step,
                                                     uint8_t* __restrict__ act,
                                                     float* __restrict__ logp,
                                                     float* __restrict__ value,
                                                     float* __restrict__ logits,
                                                     float* __restrict__ hid) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  policy_tile_f32<M, FP, H1, H2, AP, RT, DBG>(m, obs, *seedp, step, act, logp, value, logits, hid,
                                              smem, (b0 + blockIdx.x) * Shape<M, FP, H1, H2, AP, RT>::ROWS);
}

// The three layers' weights and biases in one launch (three took 2.4 us each, most of a call to
// the policy with a thousand environments: 18.3 us, and 12.3 with one): the blocks from blk0 on
// belong to the layer.
struct RepackLayer {
  const unsigned char* w_src;   // [K][N]
  const float* b_src;           // [N]
  void* w;                      // padded to Kp inputs, Np units
  float* b;
  int K, N, Kp, Np, blk0;
};
struct RepackArgs {
  RepackLayer l[3];
};
__device__ __forceinline__ const RepackLayer& repack_layer(const RepackArgs& a) {
  const int blk = blockIdx.x;
  return blk >= a.l[2].blk0 ? a.l[2] : blk >= a.l[1].blk0 ? a.l[1] : a.l[0];
}

// packed bf16 weights in MFMA fragment order: for output tile t (16 units) and k-step ks (32
// inputs), the 64 lanes' 16-byte A fragments lie back to back, lane = kq*16 + r16 holding
// W[ks*32 + kq*8 + j][t*16 + r16], j = 0..7 (zero padded). A wave's load of one fragment is
// one contiguous kilobyte, and consecutive k-steps of a tile are consecutive kilobytes. One
// fragment lane per thread.
__global__ __launch_bounds__(256) void repack_frag_k(RepackArgs args) {
  const RepackLayer& r = repack_layer(args);
  const int idx = (int)(blockIdx.x - r.blk0) * 256 + (int)threadIdx.x;
  if (idx < r.Np * r.Kp / 8) {
    const int l = idx % 64, ks = idx / 64 % (r.Kp / 32), t = idx / 64 / (r.Kp / 32);
    const int n = t * 16 + (l & 15), k = ks * 32 + (l >> 4) * 8;
    const uint16_t* src = reinterpret_cast<const uint16_t*>(r.w_src);
    uint32_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = n < r.N && k + j < r.K ? src[(size_t)(k + j) * r.N + n] : 0u;
    static_cast<uint4*>(r.w)[idx] = uint4{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16,
                                          v[6] | v[7] << 16};
  }
  if (idx < r.Np) r.b[idx] = idx < r.N ? r.b_src[idx] : 0.f;
}

// packed fp32 weights: W^T [Np][Kp], zero padded; bias fp32 [Np]
__global__ __launch_bounds__(256) void repack_f32_k(RepackArgs args) {
  const RepackLayer& r = repack_layer(args);
  const int idx = (int)(blockIdx.x - r.blk0) * 256 + (int)threadIdx.x;
  if (idx < r.Np * r.Kp) {
    const int n = idx / r.Kp, k = idx % r.Kp;
    static_cast<float*>(r.w)[idx] =
        n < r.N && k < r.K ? reinterpret_cast<const float*>(r.w_src)[(size_t)k * r.N + n] : 0.f;
  }
  if (idx < r.Np) r.b[idx] = idx < r.N ? r.b_src[idx] : 0.f;
}

// Xavier-uniform: element i of layer l takes u from the WEIGHTS block at counter
// (i, 0xFFFFFFFE, WEIGHTS<<24 | l, 0); w = (2u - 1) * lim in fp64, then fp32 (then bf16).
__global__ void init_w_k(uint64_t seed, int layer, size_t n, double lim, int bf16,
                         unsigned char* __restrict__ dst) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const u32x4 w = draw(seed, (uint32_t)i, 0xFFFFFFFEu, P_WEIGHTS, (uint32_t)layer, 0);
  const double u = unit(w.x, w.y);
  const float f = (float)((2.0 * u - 1.0) * lim);
  if (bf16) reinterpret_cast<uint16_t*>(dst)[i] = bf16_bits(f);
  else reinterpret_cast<float*>(dst)[i] = f;
}

__global__ void zero_f32_k(float* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// AC: the action count compiled into the sampler (0: m.A at run time)
template <int FP, int H1, int H2, int AP, int RT, int NW, int MINB, int TPW, bool DBG, int AC>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW * MINB / 4 > 0 ? NW * MINB / 4 : 1))) void policy_bf16_k(MlpParams m, int b0, const float* __restrict__ obs,
                                                               const uint32_t* __restrict__ obs_bf,
                                                               const uint64_t* __restrict__ seedp, uint32_t step,
                                                               uint8_t* __restrict__ act,
                                                               float* __restrict__ logp,
                                                               float* __restrict__ value,
                                                               float* __restrict__ logits,
                                                               float* __restrict__ hid) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  policy_tile_bf16<FP, H1, H2, AP, RT, NW, TPW, DBG, AC>(m, obs, obs_bf, *seedp, step, act, logp, value,
                                                       logits, hid, smem, (b0 + blockIdx.x) * (16 * RT));
}

template <bool DBG, int FP, int H1, int H2, int AP, int RT, int NW, int MINB, int TPW, int AC>
hipError_t run_policy_bf16(const MlpParams& m, const float* obs, const uint32_t* obs_bf,
                           const uint64_t* seed, uint32_t step,
                           uint8_t* act, float* logp, float* value, float* logits, float* hid,
                           EnvPart part, hipStream_t st) {
  typedef BigShape<FP, H1, H2, AP, RT, NW> Sh;
  static_assert(Sh::LDS <= 160 * 1024, "LDS budget");
  if (AC > 0 && m.A != AC) return hipErrorInvalidValue;
  auto kern = policy_bf16_k<FP, H1, H2, AP, RT, NW, MINB, TPW, DBG, AC>;
  static std::atomic<uint64_t> lds_on{0};
  const hipError_t e = allow_lds((const void*)kern, Sh::LDS, lds_on);
  if (e != hipSuccess) return e;
  if (part.e0 % Sh::ROWS != 0) return hipErrorInvalidValue;
  const dim3 grid((part.n + Sh::ROWS - 1) / Sh::ROWS), block(NW * 64);
  hipLaunchKernelGGL(kern, grid, block, Sh::LDS, st, m, part.e0 / Sh::ROWS, obs, obs_bf, seed, step, act, logp, value,
                     logits, hid);
  return hipGetLastError();
}

template <bool DBG, class M, int FP, int H1, int H2, int AP, int RT>
hipError_t run_policy(const MlpParams& m, const float* obs, const uint64_t* seed, uint32_t step,
                      uint8_t* act, float* logp, float* value, float* logits, float* hid,
                      EnvPart part, hipStream_t st) {
  typedef Shape<M, FP, H1, H2, AP, RT> Sh;
  auto kern = policy_k<M, FP, H1, H2, AP, RT, DBG>;
  static std::atomic<uint64_t> lds_on{0};
  const hipError_t e = allow_lds((const void*)kern, Sh::LDS, lds_on);
  if (e != hipSuccess) return e;
  if (part.e0 % Sh::ROWS != 0) return hipErrorInvalidValue;
  const dim3 grid((part.n + Sh::ROWS - 1) / Sh::ROWS), block(kThreads);
  hipLaunchKernelGGL(kern, grid, block, Sh::LDS, st, m, part.e0 / Sh::ROWS, obs, seed, step, act, logp, value, logits,
                     hid);
  return hipGetLastError();
}

// fp32 policy row tiles per workgroup (16 environments each): small batches take small tiles,
// so that a workgroup's serial chain of layers is short
constexpr int kF32SmallE = 4096, kF32SmallRT = 1, kF32RT = 4;

struct ShapeKey { int bf16, FP, H1, H2, AP; };
constexpr ShapeKey kShapes[] = {
    {0, 8, 64, 64, 16},      // 8-64-64-6 fp32
    {1, 32, 128, 128, 16},   // 12-128-128-6 bf16
    {1, 32, 256, 256, 32},   // 32-256-256-24(+1) bf16
    {1, 64, 256, 256, 64},   // 64-256-256-48(+1) bf16
    {1, 96, 512, 512, 112},  // 96-512-512-96(+1) bf16
};

}  // namespace

static int pad_up(int x, int m) { return (x + m - 1) / m * m; }

bool policy_shape_supported(const MlpParams& m) {
  for (const ShapeKey& s : kShapes)
    if (s.bf16 == m.bf16 && s.FP == m.FP && s.H1 == m.H1 && s.H2 == m.H2 && s.AP == m.AP)
      return true;
  return false;
}

// One bf16 shape: the configurations' own action count AC0 for that width (6K of their K)
// compiled into the sampler, any other with run-time bounds (the diagnostic instantiation
// always takes the run-time bounds; AC0 = 0 compiles none). run(ac) launches the variant.
template <bool DBG, int AC0, class Run>
static hipError_t run_shape_bf16(const MlpParams& m, Run&& run) {
  typedef std::integral_constant<int, 0> A0;
  typedef std::integral_constant<int, DBG ? 0 : AC0> AC;
  return !DBG && AC0 > 0 && m.A == AC0 ? run(AC{}) : run(A0{});
}

// Rows per workgroup (of eight waves) of the bf16 policies, by the batch. A tile's chain of
// layers is what a small batch's launch lasts, and eight waves on 16 rows make it shortest (us at
// 1024 and 8192 environments, against 32-row tiles of four waves: 12-128-128-6 5.0 and 5.4, 5.6
// and 5.8; 32-256-256-24 6.6 and 8.1, 10.5 and 10.9; 64-256-256-48 6.9 and 8.7, 12.2 and 12.4;
// 96-512-512-96 at 1024 and 4096 15.2 and 16.1, 41.8 and 42.2): up to two tiles per CU, of the 512-wide
// network, whose weights every tile reads anew, up to one. Large batches read the weights least
// often in 64-row tiles (at 28032, against 32 rows: 7.1, 8.0; 12.1, 13.1; 13.9, 15.7; 29.8, 38.8), and
// between the two 32 rows are best, up to three tiles per CU (at 16384, against 64 rows: 5.8, 6.6; in a
// rollout of 20000, per tick 29.2, 30.4) or one of the 512-wide network (8192 in a rollout: 46.5,
// 49.1; at 12032 the other way round, 20.3, 19.1).
struct Bf16Rows {
  int small_e, mid_e;
};
constexpr Bf16Rows kRows128{2 * 256 * 16, 3 * 256 * 32}, kRows256 = kRows128,
    kRows512{256 * 16, 256 * 32};

template <bool DBG>
static hipError_t launch_policy_t(const MlpParams& m, const float* obs, const uint32_t* obs_bf,
                                  const uint64_t* seed,
                                  uint32_t step, uint8_t* act, float* logp, float* value,
                                  float* logits, float* hid, EnvPart part, hipStream_t st) {
  if (!m.bf16 && m.FP == 8 && m.H1 == 64 && m.H2 == 64 && m.AP == 16)
    return m.E <= kF32SmallE
               ? run_policy<DBG, F32Mode, 8, 64, 64, 16, kF32SmallRT>(m, obs, seed, step, act, logp, value, logits, hid, part, st)
               : run_policy<DBG, F32Mode, 8, 64, 64, 16, kF32RT>(m, obs, seed, step, act, logp, value, logits, hid, part, st);
#define BSIM_BF16_ARGS (m, obs, obs_bf, seed, step, act, logp, value, logits, hid, part, st)
  if (m.bf16 && m.FP == 32 && m.H1 == 128 && m.H2 == 128 && m.AP == 16)
    return run_shape_bf16<DBG, 0>(m, [&](auto ac_v) {   // 6 measured slower
      constexpr int C = decltype(ac_v)::value;
      if (m.E <= kRows128.small_e) return run_policy_bf16<DBG, 32, 128, 128, 16, 1, 8, 1, 1, C> BSIM_BF16_ARGS;
      if (m.E <= kRows128.mid_e) return run_policy_bf16<DBG, 32, 128, 128, 16, 2, 8, 1, 1, C> BSIM_BF16_ARGS;
      return run_policy_bf16<DBG, 32, 128, 128, 16, 4, 8, 2, 1, C> BSIM_BF16_ARGS;
    });
  if (m.bf16 && m.FP == 32 && m.H1 == 256 && m.H2 == 256 && m.AP == 32)
    return run_shape_bf16<DBG, 24>(m, [&](auto ac_v) {
      constexpr int C = decltype(ac_v)::value;
      if (m.E <= kRows256.small_e) return run_policy_bf16<DBG, 32, 256, 256, 32, 1, 8, 1, 1, C> BSIM_BF16_ARGS;
      if (m.E <= kRows256.mid_e) return run_policy_bf16<DBG, 32, 256, 256, 32, 2, 8, 1, 1, C> BSIM_BF16_ARGS;
      return run_policy_bf16<DBG, 32, 256, 256, 32, 4, 8, 2, 1, C> BSIM_BF16_ARGS;
    });
  if (m.bf16 && m.FP == 64 && m.H1 == 256 && m.H2 == 256 && m.AP == 64)
    return run_shape_bf16<DBG, 48>(m, [&](auto ac_v) {
      constexpr int C = decltype(ac_v)::value;
      if (m.E <= kRows256.small_e) return run_policy_bf16<DBG, 64, 256, 256, 64, 1, 8, 1, 1, C> BSIM_BF16_ARGS;
      if (m.E <= kRows256.mid_e) return run_policy_bf16<DBG, 64, 256, 256, 64, 2, 8, 1, 1, C> BSIM_BF16_ARGS;
      return run_policy_bf16<DBG, 64, 256, 256, 64, 4, 8, 2, 1, C> BSIM_BF16_ARGS;
    });
  if (m.bf16 && m.FP == 96 && m.H1 == 512 && m.H2 == 512 && m.AP == 112)
    return run_shape_bf16<DBG, 96>(m, [&](auto ac_v) {
      constexpr int C = decltype(ac_v)::value;
      if (m.E <= kRows512.small_e) return run_policy_bf16<DBG, 96, 512, 512, 112, 1, 8, 1, 1, C> BSIM_BF16_ARGS;
      if (m.E <= kRows512.mid_e) return run_policy_bf16<DBG, 96, 512, 512, 112, 2, 8, 1, 1, C> BSIM_BF16_ARGS;
      return run_policy_bf16<DBG, 96, 512, 512, 112, 4, 8, 2, 2, C> BSIM_BF16_ARGS;
    });
#undef BSIM_BF16_ARGS
  return hipErrorInvalidValue;
}

hipError_t launch_policy(const MlpParams& m, const float* obs, const uint32_t* obs_bf,
                         const uint64_t* seed, uint32_t step, uint8_t* act, float* logp,
                         float* value, float* logits, float* hidden, EnvPart part, hipStream_t st) {
  if (obs_bf && !m.bf16) return hipErrorInvalidValue;
  if (hidden)
    return launch_policy_t<true>(m, obs, obs_bf, seed, step, act, logp, value, logits, hidden, part, st);
  return launch_policy_t<false>(m, obs, obs_bf, seed, step, act, logp, value, logits, nullptr, part, st);
}

hipError_t launch_repack(const MlpParams& m, const void* d_weights, const size_t off[6],
                         void* w1, float* b1, void* w2, float* b2, void* w3, float* b3,
                         hipStream_t st) {
  const unsigned char* src = static_cast<const unsigned char*>(d_weights);
  const int Ks[3] = {m.F, m.H1, m.H2}, Ns[3] = {m.H1, m.H2, m.Ap};
  const int Kp[3] = {m.FP, m.H1, m.H2}, Np[3] = {m.H1, m.H2, m.AP};
  void* ws[3] = {w1, w2, w3};
  float* bs[3] = {b1, b2, b3};
  RepackArgs args;
  int blocks = 0;
  for (int l = 0; l < 3; ++l) {
    args.l[l] = RepackLayer{src + off[2 * l], reinterpret_cast<const float*>(src + off[2 * l + 1]),
                            ws[l], bs[l], Ks[l], Ns[l], Kp[l], Np[l], blocks};
    // a thread per fragment lane of 8 weights, or per weight (more than there are biases: Kp >= 8)
    const int items = m.bf16 ? Np[l] * Kp[l] / 8 : Np[l] * Kp[l];
    blocks += (items + 255) / 256;
  }
  if (m.bf16) hipLaunchKernelGGL(repack_frag_k, dim3(blocks), dim3(256), 0, st, args);
  else hipLaunchKernelGGL(repack_f32_k, dim3(blocks), dim3(256), 0, st, args);
  return hipGetLastError();
}

hipError_t launch_init_weights(int F, int H1, int H2, int Ap, int bf16, uint64_t seed,
                               void* d_weights, const size_t off[6], hipStream_t st) {
  unsigned char* dst = static_cast<unsigned char*>(d_weights);
  const int dims[4] = {F, H1, H2, Ap};
  for (int l = 0; l < 3; ++l) {
    const size_t n = (size_t)dims[l] * dims[l + 1];
    const double lim = sqrt(6.0 / (double)(dims[l] + dims[l + 1]));
    hipLaunchKernelGGL(init_w_k, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, seed, l, n,
                       lim, bf16, dst + off[2 * l]);
    hipLaunchKernelGGL(zero_f32_k, dim3((dims[l + 1] + 255) / 256), dim3(256), 0, st,
                       reinterpret_cast<float*>(dst + off[2 * l + 1]), dims[l + 1]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_init_attn(uint64_t seed, void* d_weights, const size_t off[14], const int fin[7],
                            const int fout[7], hipStream_t st) {
  unsigned char* dst = static_cast<unsigned char*>(d_weights);
  for (int l = 0; l < 7; ++l) {
    const size_t n = (size_t)fin[l] * fout[l];
    const double lim = sqrt(6.0 / (double)(fin[l] + fout[l]));
    hipLaunchKernelGGL(init_w_k, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, seed, l, n,
                       lim, 0, dst + off[2 * l]);
    hipLaunchKernelGGL(zero_f32_k, dim3((fout[l] + 255) / 256), dim3(256), 0, st,
                       reinterpret_cast<float*>(dst + off[2 * l + 1]), fout[l]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace bsim
