// rollout_kernels.hip -- the fused rollouts (rollout_dev.hpp) of the 8-64-64-6 fp32 and
// 12-128-128-6 bf16 networks (any action count up to the padded width), and the choice among all.
#include "rollout_dev.hpp"

namespace bsim {
namespace {

// f(number, form) on the forms of the narrow networks for the configuration's class count
template <class F>
void narrow(const SimParams& p, const MlpParams& m, F&& f) {
  if (!m.bf16 && m.FP == 8 && m.H1 == 64 && m.H2 == 64 && m.AP == 16) {
    typedef NetF32<8, 64, 64, 16> N;
    if (p.C > 1) return;   // eight features: one server and one class
    f(0, Fused<N, 1, true>{});
    f(1, Fused<N, 1, false>{});
  }
  if (m.bf16 && m.FP == 32 && m.H1 == 128 && m.H2 == 128 && m.AP == 16) {
    if (p.C <= 2) {
      f(2, Fused<NetBf16<32, 128, 128, 16, 1, 8>, 2, true>{});
      f(3, Fused<NetBf16<32, 128, 128, 16, 1, 8>, 2, false>{});
      f(4, Fused<NetBf16<32, 128, 128, 16, 4, 8>, 2, false>{});
    } else {
      f(5, Fused<NetBf16<32, 128, 128, 16, 1, 8>, 4, true>{});
      f(6, Fused<NetBf16<32, 128, 128, 16, 1, 8>, 4, false>{});
      f(7, Fused<NetBf16<32, 128, 128, 16, 4, 8>, 4, false>{});
    }
  }
}

}  // namespace

hipError_t fused_rollout_plan(const SimParams& p, const MlpParams& m, FusedPlan* plan) {
  const hipError_t e = pick_form(p, plan, [&](auto&& f) { narrow(p, m, f); });
  return e != hipSuccess || plan->cap > 0 ? e : fused_rollout_plan_wide(p, m, plan);
}

hipError_t launch_rollout_fused(const SimParams& p, const EnvState& s, const MlpParams& m,
                                const FusedPlan& plan, uint32_t k0, int T, const RolloutOut& o,
                                hipStream_t st) {
  if (T < 1 || !o.act || plan.cap < 1) return hipErrorInvalidValue;
  if (m.bf16 && !s.obs_bf) return hipErrorInvalidValue;
  if (plan.form >= kWideForms) return launch_rollout_wide(p, s, m, plan, k0, T, o, st);
  return launch_form(p, s, m, plan, k0, T, o, st, [&](auto&& f) { narrow(p, m, f); });
}

}  // namespace bsim
