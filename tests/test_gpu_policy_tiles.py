"""The policies' tiles by batch size (16, 32 or 64 environments per workgroup of the bf16 policies;
eight lanes or one per environment of the attention policy): an environment's logits, action,
log-probability and value do not depend on the batch it is in, so batches at each size class's
edges, ragged ones among them, give the same bits as the first columns of a larger batch."""
import numpy as np
import pytest

from test_gpu_fused import bs, weights  # noqa: F401
from workloads import preset
from workloads.presets import attn_preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ATTN_SIZES = (1, 7, 1000, 40960, 40961)
SIZES = (1, 1000, 4096, 4097, 8192, 8193, 24576, 24600)


def check(bs, w, sizes, weights_of, what):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(3)
    obs = torch.randn(w["obs_dim"], max(sizes), generator=g, device="cuda")
    got = {}
    for E in sizes:
        with bs.Sim(w, n_envs=E) as sim:
            sim.reset(11)
            out = sim.policy(weights_of(sim), obs[:, :E].contiguous(), 3, want_logits=True)
            sim.sync()
            got[E] = {k: v.cpu().numpy() for k, v in out.items() if v is not None}
    big = got[max(sizes)]
    for E in sizes:
        for k, v in got[E].items():
            assert np.array_equal(v.view(np.uint8), np.ascontiguousarray(big[k][..., :E]).view(np.uint8)), \
                f"{what} E={E}: {k}"


@pytest.mark.parametrize("name,kw", [("C2", dict(value_head=1)), ("C3", {}), ("C3", dict(n_servers=3)),
                                     ("C4", {}), ("C5", dict(shadow=0))])
def test_bf16_policy_does_not_depend_on_the_batch(bs, name, kw):  # noqa: F811
    w = preset(name, **kw)
    check(bs, w, SIZES, lambda sim: sim.upload_weights(weights(w, 5)), f"{name} {kw}")


# tokens, heads, servers and units: every token count, units past one chunk and not whole chunks
@pytest.mark.parametrize("kw", [
    {}, dict(value_head=0), dict(mlp_h1=65, mlp_h2=130), dict(mlp_h1=5, mlp_h2=64, attn_heads=4),
    dict(attn_tokens=4, attn_heads=1, n_servers=2, obs_dim=16),
    dict(attn_tokens=1, n_servers=4, obs_dim=25), dict(attn_tokens=2, n_servers=4, obs_dim=24)])
def test_attention_policy_does_not_depend_on_the_batch(bs, kw):  # noqa: F811
    check(bs, attn_preset(**kw), ATTN_SIZES, lambda sim: sim.init_weights(9), f"attn {kw}")
