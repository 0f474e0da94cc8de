"""The bf16 policies' row tiles (16, 32 or 64 environments per workgroup, by batch size): an
environment's logits, action, log-probability and value do not depend on the batch it is in, so
batches at each size class's edges, ragged ones among them, give the same bits as the first
columns of a larger batch."""
import numpy as np
import pytest

from test_gpu_fused import bs, weights  # noqa: F401
from workloads import preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = (1, 1000, 4096, 4097, 8192, 8193, 24576, 24600)


@pytest.mark.parametrize("name,kw", [("C2", dict(value_head=1)), ("C3", {}), ("C3", dict(n_servers=3)),
                                     ("C4", {}), ("C5", dict(shadow=0))])
def test_policy_does_not_depend_on_the_batch(bs, name, kw):  # noqa: F811
    w = preset(name, **kw)
    g = torch.Generator(device="cuda").manual_seed(3)
    obs = torch.randn(w["obs_dim"], max(SIZES), generator=g, device="cuda")
    got = {}
    for E in SIZES:
        with bs.Sim(w, n_envs=E) as sim:
            sim.reset(11)
            out = sim.policy(sim.upload_weights(weights(w, 5)), obs[:, :E].contiguous(), 3,
                             want_logits=True)
            sim.sync()
            got[E] = {k: v.cpu().numpy() for k, v in out.items() if v is not None}
    big = got[max(SIZES)]
    for E in SIZES:
        for k, v in got[E].items():
            assert np.array_equal(v.view(np.uint8), np.ascontiguousarray(big[k][..., :E]).view(np.uint8)), \
                f"{name} {kw} E={E}: {k}"
