// rollout_wide.hip -- the fused rollouts (rollout_dev.hpp) of the 32-256-256-24 and 64-256-256-48
// bf16 networks (any action count up to the padded width).
#include "rollout_dev.hpp"

namespace bsim {
namespace {

// Weights in registers up to 32 environments per CU; from there two workgroups of four waves per
// CU that read them from L2, one's policy beside the other's tick (us per tick, 16384
// environments: 14.7 against 16.1 for one workgroup of 64 rows with the weights in registers; with
// 8 servers 28.3 against 30.4; at 8192 the other way round, 11.8 against 13.5).
template <class F>
void wide(const SimParams& p, const MlpParams& m, F&& f) {
  if (!m.bf16 || m.H1 != 256 || m.H2 != 256) return;
  if (m.FP == 32 && m.AP == 32) {
    if (p.C <= 2) {
      f(kWideForms + 0, Fused<NetBf16<32, 256, 256, 32, 1, 8>, 2, true>{});
      f(kWideForms + 1, Fused<NetBf16<32, 256, 256, 32, 1, 8>, 2, false>{});
      f(kWideForms + 2, Fused<NetBf16<32, 256, 256, 32, 2, 8>, 2, false>{});
      f(kWideForms + 3, Fused<NetBf16Stream<32, 256, 256, 32, 2, 4>, 2, false>{});
    } else {
      f(kWideForms + 4, Fused<NetBf16<32, 256, 256, 32, 1, 8>, 4, false>{});
      f(kWideForms + 5, Fused<NetBf16Stream<32, 256, 256, 32, 2, 4>, 4, false>{});
    }
  }
  if (m.FP == 64 && m.AP == 64) {
    f(kWideForms + 6, Fused<NetBf16<64, 256, 256, 64, 1, 8>, 4, true>{});
    f(kWideForms + 7, Fused<NetBf16<64, 256, 256, 64, 1, 8>, 4, false>{});
    f(kWideForms + 8, Fused<NetBf16<64, 256, 256, 64, 2, 8>, 4, false>{});
    f(kWideForms + 9, Fused<NetBf16Stream<64, 256, 256, 64, 2, 4>, 4, false>{});
  }
}

}  // namespace

hipError_t fused_rollout_plan_wide(const SimParams& p, const MlpParams& m, FusedPlan* plan) {
  return pick_form(p, plan, [&](auto&& f) { wide(p, m, f); });
}

hipError_t launch_rollout_wide(const SimParams& p, const EnvState& s, const MlpParams& m,
                               const FusedPlan& plan, uint32_t k0, int T, const RolloutOut& o,
                               hipStream_t st) {
  return launch_form(p, s, m, plan, k0, T, o, st, [&](auto&& f) { wide(p, m, f); });
}

}  // namespace bsim
