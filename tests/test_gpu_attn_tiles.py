"""The attention policy's minibatch gradient (Sec. 4.2-4.3) at the edges of its kernel's tiles:
fewer samples than a workgroup's 32 and a partial last workgroup, head widths that are not
multiples of the lanes' 8 units and that need several chunks of 64, one to eight tokens, and the
largest action count. Against the oracle with test_gpu_attn_train.py's tolerance (sums over the
samples in workgroups of 32, then 16 strided parts: no longer chains than the ones it assumes)."""
import numpy as np
import pytest

from oracle import attn as orc_attn
from test_gpu_attn_train import bs, check, logp_old_for, rand_weights, trajectory  # noqa: F401
from workloads import attn_preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [(dict(), 16), (dict(), 48), (dict(mlp_h1=65, mlp_h2=1), 80),
         (dict(mlp_h1=3, mlp_h2=200), 272), (dict(attn_tokens=1, attn_heads=1), 48),
         (dict(attn_tokens=2, attn_heads=4, mlp_h1=256, mlp_h2=130), 528),
         (dict(n_servers=4, obs_dim=24, attn_heads=4), 1040)]


@pytest.mark.parametrize("algo", [0, 1])
@pytest.mark.parametrize("over,M", CASES)
def test_attention_gradient_tiles(bs, orc, over, M, algo):  # noqa: F811
    w = attn_preset(**over)
    T, E, seed = 3, 101, 0xA78 + algo
    obs_t, act, adv, ret = trajectory(w, T, E)
    W = rand_weights(orc, w, 5)
    lp = logp_old_for(w, W, obs_t, act, 17)
    ref_loss, ref_g, ref_abs, (ti, ei) = orc_attn.minibatch_grad(
        w, W, seed, obs_t, act, lp if algo == 0 else None, adv, ret, M, algo)
    o, a, l, ad, rt = (torch.from_numpy(x).cuda() for x in (obs_t, act, lp, adv, ret))
    with bs.Sim(w, n_envs=E) as sim:
        wb = sim.upload_weights(W)
        if algo == 0:
            g, loss, idx = sim.ppo_minibatch_grad(wb, o, a, l, ad, rt, M, seed, want_index=True)
        else:
            g, loss, idx = sim.reinforce_minibatch_grad(wb, o, a, ad, rt, M, seed,
                                                        want_index=True)
        sim.sync()
        assert np.array_equal(idx.cpu().numpy(), ti * E + ei)
        check(w, sim, g, loss, ref_loss, ref_g, ref_abs, str(over))
