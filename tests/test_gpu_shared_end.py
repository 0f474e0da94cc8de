"""The learned tick's end shared among a wave's lanes (4 to 32 environments per wave, at least four
servers): an environment's observation, reward, checksum and state do not depend on the batch it
is in, so batches at every number of environments per wave give the same bits as the first
columns of a batch of 64 per wave. Server counts that do not divide over the lanes, more of them
than one read covers, and one to four classes."""
import numpy as np
import pytest

from test_gpu_fused import bs  # noqa: F401
from test_gpu_fused_forms import MIX3
from workloads import preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = (3, 4097, 9001, 17000, 40001)   # 4, 4, 8, 16 and 32 environments per wave
BIG, T = 65600, 5
CASES = [("C3", {}), ("C3", dict(MIX3, n_servers=5)), ("C4", dict(n_servers=7)),
         ("C1", dict(n_servers=16, obs_dim=72)), ("C5", dict(shadow=0, n_servers=13))]


@pytest.mark.parametrize("name,kw", CASES)
def test_tick_does_not_depend_on_the_batch(bs, name, kw):  # noqa: F811
    w = preset(name, **kw)
    g = torch.Generator(device="cuda").manual_seed(4)
    act = torch.randint(0, 6 * w["n_servers"], (T, BIG), generator=g, device="cuda", dtype=torch.uint8)
    ref = None
    for E in (BIG,) + SIZES:
        with bs.Sim(w, n_envs=E) as sim:
            sim.reset(0x5EED)
            out = [sim.step(act[t, :E].contiguous()) for t in range(T)]
            sim.sync()
            cnt, sums = sim.counters()
            got = dict(obs=torch.stack([o[0] for o in out]), rew=torch.stack([o[1] for o in out]),
                       chk=sim.checksums()[0], cnt=cnt[0], sums=sums[0])
            got = {k: v.cpu().numpy() for k, v in got.items()}
        if ref is None:
            ref = got
            continue
        for k, v in got.items():
            x = np.ascontiguousarray(ref[k][..., :E])
            assert np.array_equal(v.view(np.uint8), x.view(np.uint8)), f"{name} {kw} E={E}: {k}"
