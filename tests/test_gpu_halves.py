"""Per-tick rollouts in two chains of launches, one per half of the batch, against one chain of the
whole batch (per-launch timing on) bit for bit: at and past each size from which the halves are
taken and at those where their waves take fewer environments, with a ragged last tile in the
second half, for every policy kernel, with the value row, stored observations and the static
shadow system beside them, several times with other work on the caller's stream in between (short
such rollouts are not captured as graphs; long ones of few servers are, run by run); and inside a
caller's own capture."""
import concurrent.futures

import pytest

from test_gpu_fused import assert_same, bs, snapshot, weights  # noqa: F401
from workloads import preset
from workloads.presets import attn_preset

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    ("C1", {}, 8192, 4), ("C1", {}, 65537, 4), ("C2", dict(value_head=1), 8449, 3),
    ("C3", {}, 2048, 3), ("C3", {}, 65599, 3), ("C4", {}, 2049, 3), ("C4", {}, 8192, 3),
    ("C4", {}, 32768, 3), ("C4", {}, 65536, 2), ("C5", {}, 32768, 2), ("C5", {}, 16700, 3),
    ("attn", {}, 8200, 2), ("attn", {}, 41100, 2),
]


# the same in rollouts long enough for two chains (from 16 ticks, fewer with many
# environments and servers)
CASES += [(n, kw, E, 16 + i % 3) for i, (n, kw, E, _) in enumerate(CASES)] + [("C5", {}, 33000, 4), ("C5", {}, 65540, 2)]


@pytest.mark.parametrize("name,kw,E,T", CASES)
def test_rollout_in_halves_matches_one_chain(bs, name, kw, E, T):  # noqa: F811
    w = attn_preset(**kw) if name == "attn" else preset(name, **kw)
    ref = []
    for one_chain in (True, False):
        with bs.Sim(w, n_envs=E) as sim:
            sim.set_fused_rollout(bs.FUSE_OFF)
            sim.set_timing(one_chain)
            wb = sim.init_weights(7) if name == "attn" else sim.upload_weights(weights(w, 21))
            tr = None
            for i in range(1 if one_chain else 4):
                sim.reset(0xF0 + E)
                tr = sim.rollout(wb, T, store_obs=True, rchk=True, traj=tr)
                out = snapshot(sim, tr)
                if one_chain:
                    ref = out
                else:
                    assert_same(ref, out, f"{name} {kw} E={E}, call {i}")
                    tr.actions.zero_()
            assert one_chain or sim.graph_stats() == (0, 0)


def test_rollout_in_a_callers_capture(bs):  # noqa: F811
    w, E, T = preset("C4"), 16385, 3
    st = torch.cuda.Stream()
    with torch.cuda.stream(st), bs.Sim(w, n_envs=E) as sim:
        sim.set_fused_rollout(bs.FUSE_OFF)
        sim.set_graphs(False)
        wb = sim.upload_weights(weights(w, 21))
        sim.reset(0xCA)
        tr = sim.rollout(wb, T, store_obs=True, rchk=True)
        ref = snapshot(sim, tr)
        sim.reset(0xCA)
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
            sim.rollout(wb, T, traj=tr)
        for i in range(3):
            sim.reset(0xCA)
            for t in (tr.actions, tr.reward, tr.obs):
                t.zero_()
            g.replay()
            got = snapshot(sim, tr)
            del got["state"]   # its tick counter is the host's, which a replay does not advance
            assert_same({k: ref[k] for k in got}, got, f"replay {i}")


@pytest.mark.parametrize("name,kw,E,T", [("C1", dict(shadow=1), 8200, 300), ("C2", dict(value_head=1), 8449, 256),
                                         ("attn", {}, 8200, 130)])
def test_replayed_halves_match_one_chain(bs, name, kw, E, T):  # noqa: F811
    """Long rollouts of few servers: launched, captured and replayed run by run, with a new seed that
    only device memory carries and other device work between the replays."""
    w = attn_preset(**kw) if name == "attn" else preset(name, **kw)
    seeds, ref = (0xA1, 0xA1, 0xA2, 0xA1, 0xA2), {}
    for one_chain in (True, False):
        with bs.Sim(w, n_envs=E) as sim:
            sim.set_fused_rollout(bs.FUSE_OFF)
            sim.set_timing(one_chain)
            wb = sim.init_weights(7) if name == "attn" else sim.upload_weights(weights(w, 21))
            tr = None
            for i, seed in enumerate(seeds[1:3] if one_chain else seeds):
                sim.reset(seed)
                tr = sim.rollout(wb, T, rchk=True, traj=tr)
                out = snapshot(sim, tr)
                if i > 2:   # a ring's unused slots keep the previous episode's times
                    del out["state"]
                if one_chain:
                    ref[seed] = out
                else:
                    assert_same({k: ref[seed][k] for k in out}, out, f"{name} E={E}, call {i}")
                for t in (tr.actions, tr.reward, tr.rchk):
                    t.zero_()


@pytest.mark.parametrize("T", [17, 130])   # launched, and replayed from graphs from the third call on
def test_two_contexts_halves_from_two_threads(bs, T):  # noqa: F811
    """Two contexts, each with its own thread, stream and network, whose rollouts in halves run at the
    same time: every call's outputs are those of the context alone."""
    cases = [(preset("C1"), 8192, 0x1A), (preset("C2", value_head=1), 8449, 0x2B)]

    def calls(i, n):
        w, E, seed = cases[i]
        st = torch.cuda.Stream()
        out = []
        with torch.cuda.stream(st), bs.Sim(w, n_envs=E) as sim:
            sim.set_fused_rollout(bs.FUSE_OFF)
            wb, tr = sim.upload_weights(weights(w, 21)), None
            for _ in range(n):
                sim.reset(seed)
                tr = sim.rollout(wb, T, rchk=True, traj=tr)
                out.append(snapshot(sim, tr))
                tr.actions.zero_()
        return out

    alone = [calls(i, 1)[0] for i in range(2)]
    with concurrent.futures.ThreadPoolExecutor(2) as pool:
        jobs = [pool.submit(calls, i, 5) for i in range(2)]
        for i, job in enumerate(jobs):
            for k, out in enumerate(job.result(timeout=100)):
                assert_same(alone[i], out, f"context {i}, call {k}")
