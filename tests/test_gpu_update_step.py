"""sim_update takes Adam's step in the launch that finishes each gradient: bit for bit the
separate calls (a minibatch gradient, then adam_update with the weights rewritten), for the
networks with the four-launch gradient, one without it, and the attention policy."""
import pytest

from workloads import attn_preset, preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NETS = {"C1": preset("C1", value_head=1), "C4": preset("C4"), "C3-192": preset("C3", mlp_h2=192),
        "attn": attn_preset()}


@pytest.mark.parametrize("algo", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_update_is_gradient_and_adam(name, algo):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_05272_amd as bs
    w, T, E, M, nmb = NETS[name], 4, 200, 112, 3
    gen = torch.Generator(device="cuda").manual_seed(3)
    obs = torch.rand(T, w["obs_dim"], E, generator=gen, device="cuda")
    act = torch.randint(0, 6 * w["n_servers"], (T, E), generator=gen, device="cuda",
                        dtype=torch.uint8)
    logp = -1.0 - torch.rand(T, E, generator=gen, device="cuda")
    adv, ret = torch.randn(2, T, E, generator=gen, device="cuda", dtype=torch.float64)
    with bs.Sim(w, n_envs=E) as sim:
        got, want = [], []
        for out in (got, want):
            wb = sim.init_weights(5)
            p = sim.params_from_weights(wb)
            m, v = torch.zeros_like(p), torch.zeros_like(p)
            if out is got:
                step, losses = sim.update(wb, p, m, v, 0, obs, act, logp, adv, ret, algo, 1, nmb,
                                          M, 77, 1e-3)
                assert step == nmb
            else:
                losses = []
                for b in range(nmb):
                    seed = (77 + b * 0x9E3779B97F4A7C15) % 2 ** 64
                    if algo == bs.ALGO_PPO:
                        g, loss, _ = sim.ppo_minibatch_grad(wb, obs, act, logp, adv, ret, M, seed)
                    else:
                        g, loss, _ = sim.reinforce_minibatch_grad(wb, obs, act, adv, ret, M, seed)
                    sim.adam_update(p, g, m, v, b + 1, 1e-3, weights=wb)
                    losses.append(loss)
                losses = torch.stack(losses)
            sim.sync()
            out += [p, m, v, wb, losses]
        for a, b in zip(got, want):
            assert torch.equal(a, b)
