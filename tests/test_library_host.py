"""What the built library asks of the HIP runtime (hip_stub.py, no GPU): no kernel is launched with
more dynamic LDS than its limit on the current device allows, whatever other contexts were planned
for in between."""
import pytest

import hip_stub
from workloads import preset

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
