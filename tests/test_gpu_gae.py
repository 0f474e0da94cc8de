"""Returns / GAE (Sec. 4.3) at the edges of its kernels' tiles: the batch sizes and trajectory
lengths around the switch between the tiled and the streaming form, 16-environment tiles with a
remainder, step counts around a chunk (128 steps) and around the streaming form's groups of 8, the
batches that load one row ahead or none. All forms take the recurrence's fp64 operations in the
oracle's order, so the results are the same bits."""
import numpy as np
import pytest

from workloads import preset
from workloads.gen import seeded_rewards_values

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,T", [(1, 1), (15, 7), (16, 128), (17, 129), (33, 300), (8192, 5),
                                 (8193, 9), (14336, 3), (14352, 16), (20001, 8)])
@pytest.mark.parametrize("value", [True, False])
def test_gae_tiles(E, T, value):
    check(E, T, value)


@pytest.mark.parametrize("E,T", [(1, 63), (1, 64), (17, 72), (8192, 95), (8192, 96), (8193, 128),
                                 (14336, 119), (14336, 127), (14352, 128), (163839, 9), (163841, 9),
                                 (184304, 17), (184320, 17), (393215, 2), (393216, 3)])
@pytest.mark.parametrize("value", [True, False])
def test_gae_forms(E, T, value):
    check(E, T, value)


def check(E, T, value):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_2607_05272_amd as bs
    r, v = seeded_rewards_values(E + T, T, E, value=value)
    # an infinite and a NaN reward reach exactly the steps before them
    if E > 16:
        r[T // 2, 3] = np.inf
        r[T - 1, E - 1] = np.nan
    with bs.Sim(preset("C1", n_envs=E)) as sim:
        adv, ret = sim.returns_gae(torch.from_numpy(r).cuda(),
                                   None if v is None else torch.from_numpy(v).cuda(), 0.99, 0.95)
        sim.sync()
    ra, rr = oracle.gae(r, v, 0.99, 0.95)
    np.testing.assert_array_equal(adv.cpu().numpy(), ra)
    np.testing.assert_array_equal(ret.cpu().numpy(), rr)
