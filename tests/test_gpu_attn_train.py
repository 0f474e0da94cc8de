"""GPU parity of the attention policy's update (Sec. 4.2 network, Sec. 4.3 losses) through the
C ABI against oracle/attn.py: the REINFORCE and PPO minibatch gradients, the exact import and
export of its parameters, and the epoch x minibatch update loop.

Tolerance of a gradient entry: the GPU computes each sample's gradient terms in fp32 (chains of
at most a few dozen rounded products and sums, erf/exp/log to a few ulps, the softmax Jacobian
amplifying score errors by at most 2 in L1) and sums the M per-sample terms in a fixed order
(a sequential slice of M/256 terms, then an 8-level tree). Both errors are bounded by about 2^8 u
times the sum over samples of the magnitudes of the entry's gradient terms (u = 2^-24), which
the oracle's absolute-value backward gives; the test allows 2^-12 of that sum (16x margin). The
PPO clip decision is kept away from its boundaries: logp_old = logp_new - d with
|d - ln(1 +- clip)| >= 0.01. Loss terms: fp32 per sample, fp64 sums: 2^-12 relative."""
import math
import sys

import numpy as np
import pytest

from oracle import attn as orc_attn
from workloads import attn_preset
from workloads.gen import ppo_inputs_at, ratio_offsets, seeded_obs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CLIP = 0.2
AVOID = (np.log(1.0 - CLIP), np.log(1.0 + CLIP))
VARIANTS = {
    "paper": dict(),
    "L4_H4": dict(attn_tokens=4, attn_heads=4),
    "K2_F16": dict(n_servers=2, obs_dim=16),
}


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def bs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_05272_amd as m
    m.load()
    return m


def rand_weights(orc, w, seed):
    rng = np.random.default_rng(seed)
    return {k: (rng.standard_normal(sh) * (0.6 if k.startswith("w") else 0.2)).astype(np.float32)
            .astype(np.float64) for k, sh in orc.attn_shapes(w).items()}


def trajectory(w, T, E, seed=11):
    F, A = w["obs_dim"], 6 * w["n_servers"]
    x = seeded_obs(seed, T * E, F)
    obs_t = np.ascontiguousarray(x.reshape(T, E, F).transpose(0, 2, 1))
    tt, ee = np.meshgrid(np.arange(T), np.arange(E), indexing="ij")
    act, adv, ret = ppo_inputs_at(7, tt.astype(np.int64), ee.astype(np.int64), A)
    return obs_t, act.astype(np.uint8), adv, ret


def logp_old_for(w, W, obs_t, act, seed):
    """Old log-probabilities: the oracle's own under W minus offsets away from ln(1 +- clip)."""
    T, F, E = obs_t.shape
    A = 6 * w["n_servers"]
    x = obs_t.transpose(0, 2, 1).reshape(T * E, F).astype(np.float64)
    out = orc_attn.forward(w, W, x)["out"][:, :A]
    m = out.max(axis=1, keepdims=True)
    lse = np.log(np.exp(out - m).sum(axis=1)) + m[:, 0]
    a = act.reshape(-1).astype(np.int64)
    d = ratio_offsets(seed, T * E, avoid=AVOID)
    return (out[np.arange(T * E), a] - lse - d).astype(np.float32).reshape(T, E)


def check(w, sim, g, loss, ref_loss, ref_g, ref_abs, what):
    got = sim.unflatten_grads(g.cpu().numpy())
    worst = 0.0
    for k in ref_g:
        diff = np.abs(got[k].astype(np.float64) - ref_g[k])
        tol = 2.0 ** -12 * ref_abs[k] + 1e-30
        worst = max(worst, float((diff / tol).max()))
        assert np.all(diff <= tol), (what, k, float((diff / tol).max()))
    gl = loss.cpu().numpy()
    scale = abs(ref_loss["policy"]) + abs(ref_loss["value"]) + abs(ref_loss["entropy"])
    for i, k in enumerate(("loss", "policy", "value", "entropy")):
        assert abs(gl[i] - ref_loss[k]) <= 2.0 ** -12 * scale, (what, k)
    say(f"  {what}: max |dg| / tol {worst:.3g}")


@pytest.mark.parametrize("algo", [0, 1])
@pytest.mark.parametrize("name", sorted(VARIANTS))
def test_attention_minibatch_grad_parity(bs, orc, name, algo):
    w = attn_preset(**VARIANTS[name])
    T, E, M = 7, 300, 2048
    say(f"[attn grad] {name} algo={algo}")
    obs_t, act, adv, ret = trajectory(w, T, E)
    W = rand_weights(orc, w, 5)
    lp = logp_old_for(w, W, obs_t, act, 17) if algo == 0 else None
    seed = 0xA77 + algo
    ref_loss, ref_g, ref_abs, (ti, ei) = orc_attn.minibatch_grad(w, W, seed, obs_t, act, lp, adv,
                                                                 ret, M, algo)
    dev = torch.device("cuda")
    sim = bs.Sim(w, n_envs=E)
    wb = sim.upload_weights(W)
    o, a_, ad, rt = (torch.from_numpy(obs_t).to(dev), torch.from_numpy(act).to(dev),
                     torch.from_numpy(adv).to(dev), torch.from_numpy(ret).to(dev))
    if algo == 0:
        g, loss, idx = sim.ppo_minibatch_grad(wb, o, a_, torch.from_numpy(lp).to(dev), ad, rt, M,
                                              seed, want_index=True)
    else:
        g, loss, idx = sim.reinforce_minibatch_grad(wb, o, a_, ad, rt, M, seed, want_index=True)
    sim.sync()
    assert np.array_equal(idx.cpu().numpy(), ti * E + ei)
    check(w, sim, g, loss, ref_loss, ref_g, ref_abs, name)
    sim.close()


def test_attention_params_roundtrip(bs, orc):
    """Import gives the weights' values exactly; an Adam step with d_weights re-exports them
    as plain fp32 copies."""
    w = attn_preset()
    sim = bs.Sim(w, n_envs=64)
    W = rand_weights(orc, w, 9)
    wb = sim.upload_weights(W)
    p = sim.params_from_weights(wb)
    sim.sync()
    flat = np.concatenate([W[k].ravel() for k in orc.ATTN_KEYS])
    assert p.numel() == flat.size == sim.ppo_grad_count()
    assert np.array_equal(p.cpu().numpy().astype(np.float64), flat)
    g = torch.from_numpy(np.random.default_rng(1).standard_normal(p.numel()).astype(np.float32)).cuda()
    md, vd = torch.zeros_like(p), torch.zeros_like(p)
    sim.adam_update(p, g, md, vd, 1, 1e-3, weights=wb)
    sim.sync()
    back = bs.unpack_weights(w, wb.cpu().numpy())
    got = p.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.concatenate([back[k].ravel() for k in orc.ATTN_KEYS]), got)
    assert not np.array_equal(got, flat)
    sim.close()


@pytest.mark.parametrize("algo", [0, 1])
def test_attention_update_loop_parity(bs, orc, algo):
    """Two epochs of three minibatches with Adam (eps = 1e-2 so that each step depends smoothly
    on its gradient): the master parameters agree within steps * lr * 2^-6."""
    w = attn_preset()
    T, E = 6, 256
    epochs, nmb, M, lr, eps = 2, 3, 512, 1e-3, 1e-2
    say(f"[attn update] algo={algo}")
    obs_t, act, adv, ret = trajectory(w, T, E, seed=31)
    W = rand_weights(orc, w, 13)
    lp = logp_old_for(w, W, obs_t, act, 19)
    master = {k: v.copy() for k, v in W.items()}
    adam = dict(m={k: np.zeros_like(v) for k, v in master.items()},
                v={k: np.zeros_like(v) for k, v in master.items()}, t=0)
    ref_losses = orc_attn.update(w, master, adam, 0x5152, obs_t, act, lp, adv, ret, algo, epochs,
                                 nmb, M, lr, eps=eps)
    dev = torch.device("cuda")
    sim = bs.Sim(w, n_envs=E)
    wb = sim.upload_weights(W)
    p = sim.params_from_weights(wb)
    md, vd = torch.zeros_like(p), torch.zeros_like(p)
    step, losses = sim.update(wb, p, md, vd, 0, torch.from_numpy(obs_t).to(dev),
                              torch.from_numpy(act).to(dev), torch.from_numpy(lp).to(dev),
                              torch.from_numpy(adv).to(dev), torch.from_numpy(ret).to(dev), algo,
                              epochs, nmb, M, 0x5152, lr, eps=eps)
    sim.sync()
    assert step == epochs * nmb == adam["t"]
    ref = np.concatenate([master[k].ravel() for k in orc.ATTN_KEYS])
    got = p.cpu().numpy().astype(np.float64)
    diff = np.abs(got - ref)
    say(f"  max |dp| {diff.max():.3g} (lr {lr}, steps {step})")
    assert np.all(diff <= step * lr * 2.0 ** -6 + 2.0 ** -22 * np.abs(ref))
    gl = losses.cpu().numpy()
    scale = np.abs(ref_losses[:, 1:]).sum(axis=1)
    assert np.all(np.abs(gl - ref_losses) <= 2.0 ** -8 * scale[:, None])
    sim.close()


@pytest.mark.parametrize("name,over", [("paper", {}), ("L4_H4", VARIANTS["L4_H4"]),
                                       ("wide_heads", dict(mlp_h1=256, mlp_h2=256))])
def test_attention_logp_of_gradient_and_policy(bs, orc, name, over):
    """The gradient's log-probabilities against those stored by the policy: one sample (T = E = 1,
    advantage 1, no value and entropy terms) at its stored log-probability, so that the policy
    term is -rho = -exp(the difference). Each logit is Hp rounded products and sums of hidden units
    that are themselves D of pooled values behind a chain of some 32 operations: off by at most
    (Hp + 32) u times its magnitudes' sum S in either kernel (u = 2^-24), and a log-probability
    by twice that: a difference of 4 (Hp + 32) u S. Independent errors of that size would differ
    by sqrt of the count, so the root mean square is held to 8 sqrt(Hp + 32) u S."""
    w = attn_preset(**over)
    sim = bs.Sim(w, n_envs=1)
    sim.reset(3)
    one = torch.ones(1, 1, dtype=torch.float64, device="cuda")
    n, u, share, worst = w["mlp_h1"] + 32, 2.0 ** -24, [], 0.0
    for i in range(64):
        W = rand_weights(orc, w, 100 + i)
        x = seeded_obs(200 + i, 1, w["obs_dim"]).astype(np.float32)
        wb = sim.upload_weights(W)
        obs = torch.from_numpy(np.ascontiguousarray(x.reshape(1, -1, 1))).cuda()
        o = sim.policy(wb, obs[0], i)
        _, loss, _ = sim.ppo_minibatch_grad(wb, obs, o["actions"].view(1, 1), o["logp"].view(1, 1),
                                            one, one, 16, 5, CLIP, 0.0, 0.0)
        p = np.abs(orc_attn.forward(w, W, x.astype(np.float64))["p"][0])
        T = p @ np.abs(W["wp1"]) + np.abs(W["bp1"])
        S = (T @ np.abs(W["wp2"]) + np.abs(W["bp2"])).max()
        d = np.log(-loss.cpu().numpy()[1])
        worst = max(worst, abs(d) / (4 * n * u * S))
        share.append(d / (8 * math.sqrt(n) * u * S))
    sim.sync()
    sim.close()
    rms = float(np.sqrt(np.mean(np.square(share))))
    say(f"  {name}: max {worst:.3g}, rms {rms:.3g} of their bounds")
    assert worst <= 1.0 and rms <= 1.0
