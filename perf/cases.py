"""The workloads that this library's speed is measured on.

Each case is one call (or one short sequence of calls) that a training or evaluation program
makes through `paper_2607_05272_amd.Sim`: rollouts at the operating points of
`workloads/presets.py`, the policy and the simulator called on their own, discounted
returns / GAE, a policy-gradient minibatch and whole policy updates.

kind      one pass
rollout   reset, then T ticks of policy and simulator into the caller's trajectory buffers
policy    one batch of observations through the policy: logits, sampled actions, log-probs, value
step      reset, then T ticks under actions the caller chose (an outside policy or a replay)
gae       discounted returns / GAE over a [T][E] trajectory
grad      one minibatch gradient over a stored trajectory
update    epochs x minibatches of gradient and Adam step, weights re-exported after each

All inputs of a case are made from its seed alone. Observations are stand-ins with the ranges
of the state features (fractions in [0, 1], queue ages up to a few windows, busy flags,
zero padding is not imposed); weights are Xavier-uniform with small biases.
"""
import math

import numpy as np
import torch

import paper_2607_05272_amd as bs
from workloads import attn_preset, baseline_preset, preset

GAMMA = 0.99
CLIP, C_VALUE, C_ENTROPY = 0.2, 0.5, 0.01
LR, BETA1, BETA2, ADAM_EPS = 3e-4, 0.9, 0.999, 1e-8
ATTN_KEYS = ("w_in", "b_in", "w_qkv", "b_qkv", "w_o", "b_o", "wp1", "bp1", "wp2", "bp2",
             "wv1", "bv1", "wv2", "bv2")


# ---- cases ---------------------------------------------------------------------------------
def listed():
    return [
        # the smallest operating point (single server, fp32 policy): a REINFORCE episode batch,
        # bound by the latency of a tick
        dict(name="rollout_c1", kind="rollout", config="C1", E=256, T=1000, obs=False),
        # four servers, two classes: a mid-sized training rollout of one GPU's share
        dict(name="rollout_c3", kind="rollout", config="C3", E=16384, T=256, obs=False),
        # eight servers, bursty arrivals, observations kept for the PPO update that follows
        dict(name="rollout_c4", kind="rollout", config="C4", E=65536, T=96, obs=True),
        # the largest operating point: sixteen servers, heavy-tailed bursts, the static rule's
        # shadow system beside the learned one
        dict(name="rollout_c5", kind="rollout", config="C5", E=262144, T=96, obs=False),
        # an evaluation loop asking the policy for a ragged handful of environments at a time
        dict(name="policy_c2", kind="policy", config="C2", E=1000),
        # the simulator driven by somebody else's policy, one call per tick
        dict(name="step_c4", kind="step", config="C4", E=20000, T=16),
        # REINFORCE returns of the smallest episode batch (lambda = 1, no value head)
        dict(name="gae_c1", kind="gae", E=256, T=1000, value=False, lam=1.0),
        # GAE of a whole C4 trajectory
        dict(name="gae_c4", kind="gae", E=65536, T=1024, value=True, lam=0.95),
        # the PPO minibatch of C4 over a stored trajectory
        dict(name="grad_c4", kind="grad", config="C4", algo="ppo", E=65536, T=128, M=8192),
        # the widest network's minibatch, ragged environment count
        dict(name="grad_c5", kind="grad", config="C5", algo="ppo", E=9999, T=64, M=16384),
        # a PPO update of the C3 policy: 2 epochs x 4 minibatches
        dict(name="update_c3", kind="update", config="C3", algo="ppo", E=16384, T=128, M=4096,
             epochs=2, minibatches=4),
        # the attention policy's REINFORCE-with-baseline update
        dict(name="update_attn", kind="update", config="attn", algo="reinforce", E=16384, T=128,
             M=8192, epochs=1, minibatches=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# per configuration: environments and ticks of drawn rollouts
_ROLL = {"C1": (32, 8192, 64, 1000), "C2": (128, 16384, 64, 512), "C3": (256, 32768, 32, 256),
         "C4": (1024, 65536, 16, 96), "C5": (4096, 262144, 8, 64),
         "C3-shortest": (1024, 32768, 32, 128), "attn": (256, 262144, 32, 256)}


def draw(rng):
    kind = rng.choice(["rollout", "rollout", "rollout", "policy", "step", "gae", "grad", "grad",
                       "update"])
    if kind == "rollout":
        config = rng.choice(sorted(_ROLL))
        e0, e1, t0, t1 = _ROLL[config]
        E, T = _log(rng, e0, e1), rng.randint(t0, t1)
        return dict(kind=kind, config=config, E=E, T=T, obs=rng.random() < 0.3)
    if kind == "policy":
        return dict(kind=kind, config=rng.choice(["C1", "C2", "C3", "C4", "C5", "attn"]),
                    E=_log(rng, 16, 262144))
    if kind == "step":
        return dict(kind=kind, config=rng.choice(["C1", "C2", "C3", "C4", "C5"]),
                    E=_log(rng, 64, 131072), T=rng.randint(4, 16))
    if kind == "gae":
        value = rng.random() < 0.7
        return dict(kind=kind, E=_log(rng, 64, 65536), T=_log(rng, 64, 1024), value=value,
                    lam=0.95 if value else 1.0)
    config = rng.choice(["C1", "C3", "C4", "C5", "attn"])
    case = dict(kind=kind, config=config, algo=rng.choice(["ppo", "reinforce"]),
                E=_log(rng, 1024, 65536), T=rng.randint(32, 128), M=16 * _log(rng, 16, 1024))
    if kind == "update":
        case.update(epochs=rng.randint(1, 2), minibatches=rng.randint(2, 4))
    return case


# ---- workloads -----------------------------------------------------------------------------
def _workload(case):
    name = case["config"]
    over = dict(n_envs=case["E"])
    if case["kind"] in ("grad", "update"):
        over["value_head"] = 1       # a gradient needs the baseline output
    if name == "attn":
        return attn_preset(**over)
    if "-" in name:
        base, rule = name.split("-", 1)
        return baseline_preset(rule, base, **over)
    return preset(name, **over)


def _n_out(w):
    return 6 * w["n_servers"] + (1 if w["value_head"] else 0)


def _shapes(w):
    F, H1, H2 = w["obs_dim"], w["mlp_h1"], w["mlp_h2"]
    if w["policy_kind"] == 1:
        D, A = w["attn_embed"], 6 * w["n_servers"]
        return dict(w_in=(F, D), b_in=(D,), w_qkv=(D, 3 * D), b_qkv=(3 * D,), w_o=(D, D),
                    b_o=(D,), wp1=(D, H1), bp1=(H1,), wp2=(H1, A), bp2=(A,), wv1=(D, H2),
                    bv1=(H2,), wv2=(H2, 1), bv2=(1,))
    Ap = _n_out(w)
    return dict(w1=(F, H1), b1=(H1,), w2=(H1, H2), b2=(H2,), w3=(H2, Ap), b3=(Ap,))


def _arrays(w, seed):
    """Policy weights as fp32 numpy arrays (matrices bf16-representable in bf16 mode)."""
    rng = np.random.default_rng([seed, 1])
    out = {}
    for k, s in _shapes(w).items():
        if len(s) == 2:
            lim = math.sqrt(6.0 / (s[0] + s[1]))
            a = rng.uniform(-lim, lim, s).astype(np.float32)
            if w["mlp_bf16"]:
                a = (a.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
        else:
            a = rng.normal(0.0, 0.05, s).astype(np.float32)
        out[k] = a
    return out


def _gen(seed, k):
    return torch.Generator(device="cuda").manual_seed(seed * 16 + k)


def _observations(seed, shape, dim):
    """Observation-like fp32 values, feature axis `dim`: fractions, ages, busy flags."""
    x = torch.rand(shape, generator=_gen(seed, 2), device="cuda")
    ages = [slice(None)] * len(shape)
    ages[dim] = slice(1, None, 5)
    x[tuple(ages)] *= 3.0
    flags = [slice(None)] * len(shape)
    flags[dim] = slice(2, None, 7)
    x[tuple(flags)] = (x[tuple(flags)] > 0.5).float()
    return x


def _gae_inputs(case, seed):
    T, E = case["T"], case["E"]
    g = _gen(seed, 3)
    # throughput-like mass on some ticks minus latency-like terms
    r = torch.rand(T, E, generator=g, device="cuda", dtype=torch.float64)
    r = torch.where(r < 0.4, (r * 800.0).floor() * 1.0, torch.zeros_like(r))
    r -= torch.rand(T, E, generator=g, device="cuda", dtype=torch.float64)
    v = torch.randn(T + 1, E, generator=g, device="cuda") * 50.0 if case["value"] else None
    return r, v


def _trajectory(case, w, seed):
    """A stored trajectory: observations, actions, old log-probabilities, advantages, returns."""
    T, E, A = case["T"], case["E"], 6 * w["n_servers"]
    g = _gen(seed, 4)
    return dict(
        obs=_observations(seed, (T, w["obs_dim"], E), 1),
        act=torch.randint(0, A, (T, E), generator=g, device="cuda", dtype=torch.uint8),
        # near the log-probability of a nearly uniform policy, so that ratios lie on both
        # sides of the clip range
        logp=-math.log(A) + 0.4 * torch.randn(T, E, generator=g, device="cuda"),
        adv=torch.randn(T, E, generator=g, device="cuda", dtype=torch.float64),
        ret=torch.randn(T, E, generator=g, device="cuda", dtype=torch.float64))


def prepare(case, seed):
    s = dict(case=case, seed=seed)
    kind, E, T = case["kind"], case["E"], case.get("T")
    if kind == "gae":
        # the context is the one of the rollout whose rewards these are (any shape will do)
        w = preset("C1", n_envs=E)
        s["sim"] = bs.Sim(w)
        s["r"], s["v"] = _gae_inputs(case, seed)
        s["adv"], s["ret"] = torch.empty_like(s["r"]), torch.empty_like(s["r"])
        return s
    w = _workload(case)
    s["sim"] = sim = bs.Sim(w)
    if kind == "step":
        g = _gen(seed, 5)
        s["actions"] = torch.randint(0, 6 * w["n_servers"], (T, E), generator=g, device="cuda",
                                     dtype=torch.uint8)
        return s
    s["wb"] = sim.upload_weights(_arrays(w, seed))
    if kind == "rollout":
        s["traj"] = bs.Trajectory(T, E, w["obs_dim"], "cuda", value=bool(w["value_head"]),
                                  shadow=bool(w["shadow"]), obs=case["obs"])
    elif kind == "policy":
        sim.reset(seed)
        s["obs"] = _observations(seed, (w["obs_dim"], E), 0)
    else:
        s["tr"] = _trajectory(case, w, seed)
        if kind == "update":
            s["params"] = sim.params_from_weights(s["wb"])
            s["m"], s["v"] = torch.zeros_like(s["params"]), torch.zeros_like(s["params"])
            s["step"] = 0
        else:
            s["grads"] = torch.empty(sim.ppo_grad_count(), dtype=torch.float32, device="cuda")
            s["loss"] = torch.empty(4, dtype=torch.float64, device="cuda")
    return s


def run(s):
    case, sim, seed = s["case"], s["sim"], s["seed"]
    kind = case["kind"]
    if kind == "rollout":
        sim.reset(seed)
        tr = sim.rollout(s["wb"], case["T"], traj=s["traj"])
        return {k: getattr(tr, k) for k in ("actions", "logp", "reward", "reward_shadow", "value",
                                            "obs")}
    if kind == "policy":
        return sim.policy(s["wb"], s["obs"], 0, want_logits=True)
    if kind == "step":
        sim.reset(seed)
        return [sim.step(a) for a in s["actions"]]
    if kind == "gae":
        return sim.returns_gae(s["r"], s["v"], GAMMA, case["lam"], s["adv"], s["ret"])
    tr = s["tr"]
    if kind == "grad":
        if case["algo"] == "ppo":
            g, loss, _ = sim.ppo_minibatch_grad(s["wb"], tr["obs"], tr["act"], tr["logp"],
                                                tr["adv"], tr["ret"], case["M"], seed, CLIP,
                                                C_VALUE, C_ENTROPY, grads=s["grads"],
                                                loss=s["loss"])
        else:
            g, loss, _ = sim.reinforce_minibatch_grad(s["wb"], tr["obs"], tr["act"], tr["adv"],
                                                      tr["ret"], case["M"], seed, C_VALUE,
                                                      C_ENTROPY, grads=s["grads"], loss=s["loss"])
        return dict(loss=loss, grads=g)
    algo = bs.ALGO_PPO if case["algo"] == "ppo" else bs.ALGO_REINFORCE
    s["step"], losses = sim.update(s["wb"], s["params"], s["m"], s["v"], s["step"], tr["obs"],
                                   tr["act"], tr["logp"], tr["adv"], tr["ret"], algo,
                                   case["epochs"], case["minibatches"], case["M"], seed, LR, CLIP,
                                   C_VALUE, C_ENTROPY, BETA1, BETA2, ADAM_EPS)
    return dict(losses=losses, params=s["params"], m=s["m"], v=s["v"])


# ---- work and tolerances -------------------------------------------------------------------
def _policy_flops(w):
    F, H1, H2 = w["obs_dim"], w["mlp_h1"], w["mlp_h2"]
    if w["policy_kind"] == 1:
        L, D, A = w["attn_tokens"], w["attn_embed"], 6 * w["n_servers"]
        dh = D // w["attn_heads"]
        return 2 * (F * D + L * D * 3 * D + 2 * w["attn_heads"] * L * L * dh + L * D * D + D * H1
                    + H1 * A + (D * H2 + H2 if w["value_head"] else 0))
    return 2 * (F * H1 + H1 * H2 + H2 * _n_out(w))


def _n_params(w):
    return sum(int(np.prod(s)) for s in _shapes(w).values())


def work(case):
    kind, E, T = case["kind"], case["E"], case.get("T", 1)
    if kind == "gae":
        return dict(bytes=T * E * (24 + (4 if case["value"] else 0)), flops=6 * T * E)
    w = _workload(case)
    P, F = _n_params(w), w["obs_dim"]
    wbytes = P * (2 if w["mlp_bf16"] else 4)
    if kind == "rollout":
        row = 1 + 4 + 8 + (4 if w["value_head"] else 0) + (8 if w["shadow"] else 0)
        row += 4 * F if case["obs"] else 0
        return dict(bytes=wbytes + T * E * row, flops=T * E * _policy_flops(w))
    if kind == "policy":
        return dict(bytes=wbytes + E * (4 * F + 4 * _n_out(w) + 9), flops=E * _policy_flops(w))
    if kind == "step":
        return dict(bytes=T * E * (1 + 4 * F + 8 + (8 if w["shadow"] else 0)), flops=0)
    # forward, backward through the activations and the weight products
    n = case["M"] * (case["epochs"] * case["minibatches"] if kind == "update" else 1)
    flops = n * 3 * _policy_flops(w)
    if w["policy_kind"] == 0:
        flops -= n * 2 * F * w["mlp_h1"]
    moved = n * (4 * F + 1 + 4 + 16)
    if kind == "grad":
        return dict(bytes=moved + wbytes + 4 * P, flops=flops)
    return dict(bytes=moved + n // case["M"] * (2 * wbytes + 6 * 4 * P), flops=flops)


def tolerance(case):
    kind = case["kind"]
    if kind in ("rollout", "step"):
        # a rollout is one course of discrete events: the same seed gives the same course, and
        # an action sampled differently sends its environment down another one
        return "exact"
    if kind == "gae":
        return dict(rel=1e-13, max=1e-12)    # the same fp64 recurrence in another association
    # four times what the hidden units' order changes (the same sums in another order): fp32
    # networks by rounding alone, bf16 ones because a hidden activation near a rounding boundary
    # moves by one bf16 step; an update carries that through its Adam steps
    if not _workload(case)["mlp_bf16"]:
        return dict(rel=2e-6, max=4e-5, differ=1e-4)
    if kind == "policy":
        return dict(rel=2.5e-4, max=2e-2, differ=1e-4)
    if kind == "grad":
        return dict(rel=5e-5, max=4e-3)
    return dict(rel=1.2e-3, max=4e-2)


# ---- the same in 64 bits -------------------------------------------------------------------
def _bf16(x):
    return x.float().bfloat16().double()


class _RoundBf16(torch.autograd.Function):
    """The policy's rounding of a layer's input to bf16; its gradient passes through."""

    @staticmethod
    def forward(ctx, x):
        return _bf16(x)

    @staticmethod
    def backward(ctx, g):
        return g


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x * math.sqrt(0.5)))


def _forward(w, p, x):
    """Logits [n][A] and value [n] (or None) of observations x [n][F], parameters p."""
    A = 6 * w["n_servers"]
    if w["policy_kind"] == 1:
        L, D, NH = w["attn_tokens"], w["attn_embed"], w["attn_heads"]
        n, F = x.shape
        dh = D // NH
        tok = (x.view(n, L, F // L, 1) * p["w_in"].view(1, L, F // L, D)).sum(2) + p["b_in"]
        q, k, v = ((tok.reshape(n * L, D) @ p["w_qkv"] + p["b_qkv"]).view(n, L, 3, NH, dh)
                   .unbind(2))
        sc = (q.unsqueeze(2) * k.unsqueeze(1)).sum(-1) / math.sqrt(dh)      # [n][L][L][NH]
        o = (torch.softmax(sc, 2).unsqueeze(-1) * v.unsqueeze(1)).sum(2).reshape(n, L, D)
        pool = o.mean(1) @ p["w_o"] + p["b_o"]
        lg = _gelu(pool @ p["wp1"] + p["bp1"]) @ p["wp2"] + p["bp2"]
        V = (_gelu(pool @ p["wv1"] + p["bv1"]) @ p["wv2"] + p["bv2"]).squeeze(1)
        return lg, V if w["value_head"] else None
    rnd = _RoundBf16.apply if w["mlp_bf16"] else (lambda t: t)
    h = rnd(_gelu(rnd(x) @ p["w1"] + p["b1"]))
    h = rnd(_gelu(h @ p["w2"] + p["b2"]))
    out = h @ p["w3"] + p["b3"]
    return out[:, :A], out[:, A] if w["value_head"] else None


def _params64(w, seed):
    return {k: torch.from_numpy(a).cuda().double() for k, a in _arrays(w, seed).items()}


def _sample_index(seed, M, n):
    """The minibatch's positions floor(u n): u from the Philox4x32-10 block (Salmon et al. 2011)
    at counter (m, 0xFFFFFFFD, 6 << 24, 0) under the 64-bit key `seed`, top 53 bits centred."""
    u64 = np.uint64
    lo32 = u64(0xFFFFFFFF)
    c = [np.arange(M, dtype=u64), np.full(M, 0xFFFFFFFD, u64), np.full(M, 6 << 24, u64),
         np.zeros(M, u64)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = u64(0xD2511F53) * c[0], u64(0xCD9E8D57) * c[2]
        c = [(p1 >> u64(32)) ^ c[1] ^ u64(k0), p1 & lo32, (p0 >> u64(32)) ^ c[3] ^ u64(k1),
             p0 & lo32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    v = ((c[1] << u64(32)) | c[0]) >> u64(11)
    i = np.floor((v.astype(np.float64) + 0.5) * 2.0 ** -53 * float(n)).astype(np.int64)
    return torch.from_numpy(np.minimum(i, n - 1)).cuda()


def _grads(case, w, p, tr, seed):
    """(flat gradient, loss terms) of one minibatch at parameters p."""
    M, E = case["M"], case["E"]
    i = _sample_index(seed, M, case["T"] * E)
    t, e = i // E, i % E
    x = tr["obs"][t, :, e].double()
    act, adv, ret = tr["act"][t, e].long(), tr["adv"][t, e], tr["ret"][t, e]
    p = {k: a.clone().requires_grad_(True) for k, a in p.items()}
    lg, V = _forward(w, p, x)
    lp = torch.log_softmax(lg, 1)
    la = lp.gather(1, act[:, None]).squeeze(1)
    if case["algo"] == "ppo":
        rho = torch.exp(la - tr["logp"][t, e].double())
        pi = -torch.minimum(rho * adv, rho.clamp(1 - CLIP, 1 + CLIP) * adv).mean()
    else:
        pi = -(adv * la).mean()
    vl = C_VALUE * ((V - ret) ** 2).mean()
    ent = C_ENTROPY * (lp.exp() * lp).sum(1).mean()
    loss = pi + vl + ent
    loss.backward()
    flat = torch.cat([p[k].grad.reshape(-1) for k in _shapes(w)])
    return flat, torch.stack([loss, pi, vl, ent]).detach()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("rollout", "step"):
        return None          # a course of discrete events, compared bit for bit
    if kind == "gae":
        r, v = _gae_inputs(case, seed)
        v = v.double() if v is not None else torch.zeros(r.shape[0] + 1, r.shape[1],
                                                         dtype=torch.float64, device="cuda")
        adv, ret, a = torch.empty_like(r), torch.empty_like(r), torch.zeros_like(r[0])
        gl = GAMMA * case["lam"]
        for t in range(case["T"] - 1, -1, -1):
            a = (r[t] + GAMMA * v[t + 1]) - v[t] + gl * a
            adv[t] = a
            ret[t] = a + v[t]
        return adv, ret
    w = _workload(case)
    p = _params64(w, seed)
    if kind == "policy":
        lg, V = _forward(w, p, _observations(seed, (w["obs_dim"], case["E"]), 0).t().double())
        # the sampled action turns on which side of a boundary a rounded sum falls
        out = lg if V is None else torch.cat([lg, V[:, None]], 1)
        return dict(actions=None, logp=None, value=V, logits=out.t())
    tr = _trajectory(case, w, seed)
    if kind == "grad":
        g, loss = _grads(case, w, p, tr, seed)
        return dict(loss=loss, grads=g)
    # the update: master parameters in 64 bits, the policy's weights rounded from them
    keys = list(_shapes(w))
    sizes = [a.numel() for a in p.values()]
    flat = torch.cat([p[k].reshape(-1) for k in keys])
    m, v, losses = torch.zeros_like(flat), torch.zeros_like(flat), []
    for b in range(case["epochs"] * case["minibatches"]):
        key = (seed + b * 0x9E3779B97F4A7C15) & 0xFFFFFFFFFFFFFFFF
        parts = torch.split(flat, sizes)
        cur = {k: (_bf16(a) if w["mlp_bf16"] and p[k].dim() == 2 else a).reshape(p[k].shape)
               for k, a in zip(keys, parts)}
        g, loss = _grads(case, w, cur, tr, key)
        losses.append(loss)
        m = BETA1 * m + (1 - BETA1) * g
        v = BETA2 * v + (1 - BETA2) * g * g
        flat = flat - LR * (m / (1 - BETA1 ** (b + 1))) / (
            torch.sqrt(v / (1 - BETA2 ** (b + 1))) + ADAM_EPS)
    return dict(losses=torch.stack(losses), params=flat, m=m, v=v)
