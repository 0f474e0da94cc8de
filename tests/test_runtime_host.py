"""The host runtime's launch sequences (csrc/runtime.cpp linked with the recording stand-ins of
runtime_stub.cpp, no GPU): a rollout that fails in the middle of its two chains still joins
every stream it forked back to the caller's; the second stream is made when a rollout needs it; a
repeated rollout in halves is replayed from graphs; short rollouts take neither a second chain nor
a second round of fused workgroups."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2607_05272_amd import _lib as L
from workloads.presets import attn_preset, preset

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CALLER = 1000   # the caller's stream handle


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    csrc = os.path.join(ROOT, "paper_2607_05272_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", "/opt/rocm/include", "-I", csrc, "-I", os.path.join(ROOT, "include"),
                    os.path.join(csrc, "runtime.cpp"), os.path.join(HERE, "runtime_stub.cpp"),
                    "-Wl,-Bsymbolic", "-o", out], check=True)
    lib = C.CDLL(out)
    lib.stub_log.restype = C.c_char_p
    return lib


class Ctx:
    """A context over the stand-ins; rollout() returns (status, log lines split into words)."""

    def __init__(self, lib, w, n_envs, fused_cap=0):
        self.lib, self.cap = lib, fused_cap
        self.cfg = L.make_cfg(w, n_envs)
        self.h = C.c_void_p()
        lib.stub_reset(-1, fused_cap)
        assert lib.sim_create(C.byref(self.cfg), C.c_void_p(CALLER), C.byref(self.h)) == 0
        self.created = self.log()
        assert lib.sim_reset(self.h, C.c_uint64(1)) == 0
        fields = ["actions", "logp", "reward"] + (["reward_shadow"] if w["shadow"] else []) + \
            (["value"] if w["value_head"] else [])
        self.traj = L.SimTraj(**{f: (i + 1) << 40 for i, f in enumerate(fields)})

    def log(self):
        return [l.split() for l in self.lib.stub_log().decode().splitlines()]

    def rollout(self, T, fail_after=-1, reset=True):
        if reset:
            assert self.lib.sim_reset(self.h, C.c_uint64(1)) == 0
        self.lib.stub_reset(fail_after, self.cap)
        rc = self.lib.sim_rollout(self.h, C.c_void_p(1 << 50), T, C.byref(self.traj))
        return rc, self.log()


def launches(log, kind):
    return [l for l in log if l[0] == "launch" and l[2] == kind]


def joined(log, s, after):
    """Whether the caller's stream waits, directly or over others, for what s holds at `after`."""
    return any(l[0] == "wait" and l[2] == ev and (l[1] == str(CALLER) or joined(log, l[1], j))
               for i, ev in [(i, l[2]) for i, l in enumerate(log) if i > after and l[:2] == ["record", s]]
               for j, l in enumerate(log) if j > i)


def assert_joined(log):
    for s in {l[1] for l in log if l[0] in ("launch", "graph")} - {str(CALLER)}:
        last = max(i for i, l in enumerate(log) if l[0] in ("launch", "graph") and l[1] == s)
        assert joined(log, s, last), f"stream {s} is not joined: {log[last:]}"


@pytest.mark.parametrize("name,n", [("C4", 65536), ("C5", 65536)])
def test_failed_rollout_joins_its_streams(stub, name, n):
    x = Ctx(stub, preset(name), n)
    assert stub.sim_set_graphs(x.h, 0) == 0
    rc, log = x.rollout(8)
    assert rc == 0 and {l[3] for l in launches(log, "step")} == {"0", "32768"}
    assert_joined(log)
    total = sum(l[0] == "launch" for l in log)
    for k in range(total):
        rc, log = x.rollout(8, fail_after=k)
        assert rc == -3
        assert_joined(log)
    # the same of a replay (three servers at most): its launches are the head's and the first policy
    x = Ctx(stub, preset(name, n_servers=3), 32768)
    x.rollout(128)
    rc, log = x.rollout(128)
    assert rc == 0 and [l for l in log if l[0] == "graph"]
    for k in range(sum(l[0] == "launch" for l in log)):
        rc, log = x.rollout(128, fail_after=k)
        assert rc == -3
        assert_joined(log)


def test_second_stream_only_for_rollouts_in_halves(stub):
    x = Ctx(stub, preset("C4"), 65536)
    assert not [l for l in x.created if l[0] == "stream"]   # a context may never roll out in halves
    rc, log = x.rollout(64)
    assert rc == 0 and len([l for l in log if l[0] == "stream"]) == 1
    rc, log = x.rollout(65)
    assert rc == 0 and not [l for l in log if l[0] == "stream"]


@pytest.mark.parametrize("w,n,T", [(preset("C2"), 40000, 600), (preset("C1"), 40000, 256),
                                   (attn_preset(), 40960, 256),
                                   (preset("C3", n_servers=2, obs_dim=18), 36864, 128)])
def test_repeated_rollout_in_halves_is_replayed(stub, w, n, T):
    x = Ctx(stub, w, n)
    rc, first = x.rollout(T)
    assert rc == 0 and not [l for l in first if l[0] == "graph"]
    per_chain = 2 * T + (1 if w["value_head"] else 0)
    for i in range(3):   # captured and replayed, then replayed
        rc, log = x.rollout(T)
        assert rc == 0
        assert_joined(log)
        # the host's part no longer grows with every tick's launches
        assert len([l for l in log if l[0] == "launch"]) <= 4
        g = [l for l in log if l[0] == "graph"]
        assert len(g) == 2 * -(-per_chain // 512)   # 256 ticks each
        assert all(a[1] != b[1] for a, b in zip(g, g[1:])), "the chains' graphs take turns"
        first_policy = len(launches(log, "policy"))
        assert sum(int(l[2]) for l in g) + first_policy == 2 * per_chain and first_policy == 1
    # another length is launched again
    rc, log = x.rollout(T + 1)
    assert rc == 0 and not [l for l in log if l[0] == "graph"]


@pytest.mark.parametrize("w,n,T,chains", [
    (preset("C1"), 65536, 1, 1), (preset("C1"), 65536, 15, 1), (preset("C1"), 65536, 16, 2),
    (attn_preset(), 65536, 8, 1), (attn_preset(), 262144, 4, 2), (preset("C4"), 32768, 15, 1), (preset("C4"), 32768, 16, 2),
    (preset("C5"), 32768, 3, 1), (preset("C5"), 32768, 4, 2), (preset("C5"), 32767, 4, 1),
    (preset("C5"), 65536, 2, 2)])
def test_short_rollouts_are_one_chain(stub, w, n, T, chains):
    x = Ctx(stub, w, n)
    for i in range(3):
        rc, log = x.rollout(T)
        assert rc == 0 and not [l for l in log if l[0] == "graph"]
        assert len(launches(log, "step")) == chains * T
        forks = len([l for l in log if l[0] == "record"])
        assert forks == (2 if chains == 2 else 0) + (2 if w["shadow"] else 0)


@pytest.mark.parametrize("w,n,fused_from", [(preset("C1"), 8192, 1), (preset("C1"), 8193, 4),
                                            (preset("C1"), 16384, 4), (preset("C1"), 16385, None),
                                            (preset("C3"), 12288, 4), (preset("C4"), 8193, None)])
def test_a_second_round_is_for_more_than_a_few_ticks(stub, w, n, fused_from):
    x = Ctx(stub, w, n, fused_cap=8192)
    for T in (1, 3, 4, 200):
        rc, log = x.rollout(T)
        assert rc == 0
        assert bool(launches(log, "fused")) == (fused_from is not None and T >= fused_from)
