"""What the built library asks of the HIP runtime (hip_stub.py, no GPU): no kernel is launched with
more dynamic LDS than its limit on the current device allows, whatever other contexts were planned
for in between."""
import pytest

import hip_stub
from workloads import attn_preset, preset

P = 1 << 40   # a device pointer (nothing reads it)


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hip_stub.build(str(tmp_path_factory.mktemp("stub") / "libhipstub.so"))


def assert_lds_allowed(log):
    n = 0
    for l in log:
        if l[0] == "launch" and int(l[8]) > 64 * 1024:
            n += 1
            assert int(l[8]) <= int(l[9]), f"{l[1]}: {l[8]} bytes of LDS, limit {l[9]}"
    return n


def test_lds_limits_with_contexts_between(stub):
    roll = lambda c: dict(call="sim_rollout", ctx=c, args=[P, 4, "traj"])   # noqa: E731
    new = lambda n, **kw: dict(new=n, w=preset("C4", **kw), n_envs=64)      # noqa: E731
    out = hip_stub.run(stub, [new("long", queue_cap=100), roll("long"),
                              new("short", queue_cap=5), roll("short"), roll("long")])
    assert all(rc == 0 for rc, _ in out)
    assert [assert_lds_allowed(log) for _, log in out] == [0, 1, 0, 0, 1]


@pytest.mark.parametrize("call", [
    dict(call="sim_policy", ctx="a", args=[P, P, 0, P, P, P, P]),
    dict(call="sim_rollout", ctx="a", args=[P, 4, "traj"]),
    dict(call="ppo_minibatch_grad", ctx="a", args=[P, 4, P, P, P, P, P, 8192, 1, 0.2, 0.5, 0.01, P, P, None])])
def test_lds_limits_on_another_device(stub, call):
    out = hip_stub.run(stub, [x for d in (0, 1)
                              for x in (dict(device=d), dict(new="a", w=preset("C5"), n_envs=40000), call)])
    assert all(rc == 0 for rc, _ in out)
    first, second = [assert_lds_allowed(out[i][1]) for i in (2, 5)]
    assert first == second > 0


def grad(c, M, name="ppo_minibatch_grad"):
    return dict(call=name, ctx=c, args=[P, 4, P, P, P, P, P, M, 1, 0.2, 0.5, 0.01, P, P, None])


@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4", "C5"])
def test_rollout_networks_gradients_take_four_launches(stub, name):
    """From the smallest minibatch on, in the scratch that this form uses."""
    w = preset(name, value_head=1)
    F, H1, H2, A = (-(-x // 64) * 64 for x in (w["obs_dim"], w["mlp_h1"], w["mlp_h2"],
                                               6 * w["n_servers"] + 1))
    e, two = (2, 2) if w["mlp_bf16"] else (4, 1)
    for M in (16, 32, 48, 64, 80, 4096, 8192, 16384):
        out = hip_stub.run(stub, [dict(new="a", w=w, n_envs=4096), grad("a", M)])
        assert all(rc == 0 for rc, _ in out)
        log = out[1][1]
        names = [l[1] for l in log if l[0] == "launch"]
        assert len(names) == 4 and "pg_mlp_k" in names[1], f"M = {M}: {names}"
        # x twice, both activations, the gradients' terms and 32 bytes per sample; partial sums
        Mp = -(-M // 64) * 64
        per = e * (2 * F + H1 + H2 + two * (A + H2 + H1)) + 32 + 4 * (A + H2 + H1) // 16
        (size,) = [int(l[1]) for l in log if l[0] == "malloc"]
        assert size <= Mp * per + (8 << 20)


def test_noalloc_limit_stays(stub):
    """The no-allocation entry point's limit is the one that batchsim.h states."""
    w = preset("C4")
    for M, rc in ((8192, 0), (16384, -1)):
        out = hip_stub.run(stub, [dict(new="a", w=w, n_envs=512), grad("a", M, "ppo_minibatch_grad_noalloc")])
        assert out[1][0] == rc and not [l for l in out[1][1] if l[0] == "malloc"]


def test_attention_gradient_scratch(stub):
    """A row of partial sums and three loss terms per 32 samples; the no-allocation entry's limit of
    4 M P + 24 M bytes stays."""
    w = attn_preset()
    n = 8 * 4 + 4 + 4 * 12 + 12 + 4 * 4 + 4 + 4 * 64 + 64 + 64 * 6 + 6 + 4 * 64 + 64 + 64 + 1
    for M in (16, 48, 8192):
        out = hip_stub.run(stub, [dict(new="a", w=w, n_envs=512), grad("a", M)])
        assert out[1][0] == 0
        assert [int(l[1]) for l in out[1][1] if l[0] == "malloc"] == [-(-M // 32) * (4 * n + 24)]
    M = ((96 << 20) // (4 * n + 24)) // 16 * 16
    for m, rc in ((M, 0), (M + 16, -1)):
        out = hip_stub.run(stub, [dict(new="a", w=w, n_envs=512), grad("a", m, "ppo_minibatch_grad_noalloc")])
        assert out[1][0] == rc
