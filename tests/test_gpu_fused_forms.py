"""The fused rollout's forms (which tile, weights in registers or from L2, request rings in LDS or in
memory) at the edges of what each takes, against the per-tick launches bit for bit: batches
just past what the smaller tile holds at once, one environment, queues too long for LDS, the
largest server count of each padded width, three classes, more workgroups than are resident at
once, and few ticks in a row."""
import pytest

from test_gpu_fused import assert_same, bs, snapshot, weights  # noqa: F401
from workloads import preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIX3 = dict(n_classes=3, class_mix=[0.5, 0.3, 0.2], service_kind=[1, 0, 2],
            svc_alpha=[0.0, 2e-3, 1e-3], svc_beta=[1e-4] * 3, svc_median=[1e-3, 0.0, 0.0],
            svc_sigma=1.0, w_class=[200.0, 100.0, 20.0])
CASES = [
    ("C1", {}, 1, 9), ("C1", {}, 4097, 5), ("C1", dict(queue_cap=255, rates=[20000.0]), 3000, 12),
    ("C2", dict(n_servers=2, obs_dim=18, value_head=1), 77, 12), ("C2", {}, 4100, 5),
    ("C2", dict(MIX3, queue_cap=255, obs_dim=14), 300, 12),
    ("C3", dict(n_servers=5), 4096, 4), ("C3", {}, 4111, 4), ("C3", {}, 9001, 3),
    ("C3", dict(MIX3, n_servers=4), 4300, 4), ("C3", dict(queue_cap=255), 500, 8),
    ("C4", dict(n_servers=10), 129, 5), ("C4", {}, 4099, 3), ("C4", {}, 8300, 3),
    ("C4", dict(queue_cap=255, rates=[40000.0] * 3), 64, 12),
    ("C1", {}, 16401, 3), ("C2", {}, 16401, 3), ("C3", {}, 32769, 2),   # two rounds and a third
]


@pytest.mark.parametrize("name,kw,E,T", CASES)
def test_fused_forms_match_per_tick(bs, name, kw, E, T):  # noqa: F811
    w = preset(name, **kw)
    out = []
    for mode in (bs.FUSE_OFF, bs.FUSE_ON):
        with bs.Sim(w, n_envs=E) as sim:
            sim.set_fused_rollout(mode)
            sim.set_graphs(False)
            sim.reset(0xF0 + E)
            wb = sim.upload_weights(weights(w, 21))
            out.append([snapshot(sim, sim.rollout(wb, t, store_obs=t == T, rchk=True))
                        for t in (T, 1, T)])
    for i, (a, b) in enumerate(zip(*out)):
        assert_same(a, b, f"{name} {kw} E={E}, call {i}")


def test_contexts_with_other_queues_between(bs):  # noqa: F811
    """Two contexts of one network whose rings take different shares of LDS, rolled out in turn."""
    w = {"long": preset("C4", queue_cap=100), "short": preset("C4", queue_cap=5)}
    out = []
    for mode in (bs.FUSE_OFF, bs.FUSE_ON):
        with bs.Sim(w["long"], n_envs=64) as a, bs.Sim(w["short"], n_envs=64) as b:
            got = []
            for sim, k in ((a, "long"), (b, "short"), (a, "long"), (b, "short")):
                sim.set_fused_rollout(mode)
                sim.set_graphs(False)
                sim.reset(0xAB)
                wb = sim.upload_weights(weights(w[k], 21))
                got.append(snapshot(sim, sim.rollout(wb, 6, rchk=True)))
            out.append(got)
    for i, (x, y) in enumerate(zip(*out)):
        assert_same(x, y, f"rollout {i}")
