"""The minibatch gradient (Sec. 4.3) at the edges of its kernels' tiles, for every network with
the four-launch form and one without: the smallest minibatch, row padding (48 and 80 samples in
64-sample blocks), the switch from 16 to 32 samples per workgroup (4096, 4112) with a partial
last workgroup, chunks of the weight product that do not divide the steps, and fewer actions
than the network's padded width. Against the numpy oracle with test_gpu_ppo.py's tolerances,
which are derived there for M <= 4096; at 4112 samples the same bounds hold (sqrt(M) u)."""
import pytest

from test_gpu_ppo import bs, run_small, workload  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [("C1", {}, 16), ("C1", {}, 80), ("C2", {}, 48), ("C2", {}, 4112), ("C3", {}, 80),
         ("C3", dict(n_servers=2, obs_dim=18), 1040), ("C3", dict(mlp_h1=192), 272),
         ("C4", {}, 16), ("C4", {}, 4112), ("C5", {}, 48), ("C5", {}, 4112)]


@pytest.mark.parametrize("name,over,M", CASES)
def test_minibatch_tiles(bs, name, over, M):  # noqa: F811
    run_small(bs, workload(name, **over), 5, 333, M, seed=0xC0FFEE + M)
