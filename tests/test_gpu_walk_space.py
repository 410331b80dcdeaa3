"""The space of the walk's hand-down lists beyond what 32-bit offsets reach.

A pair list of more than 2^30 entries gives the lists a buffer of more than 2^31 words
(that list's buffer is theirs where the queue is smaller); they may use it only up to
there.  The lists found and the sums over them are those of the default capacities, bit
for bit."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import run_collide, run_gravity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


# long lists: a small opening angle over small leaves
OVER = dict(leaf_size=2, theta_min=0.25, ncs=0, ncc_pre=0, ncc_post=0, m2l_per_cell=8192,
            p2p_per_leaf=8192)


@pytest.mark.parametrize("capacity", [1_300_000_000, (1 << 31) + 10])
def test_large_pair_capacity_keeps_every_list(nc, orc, capacity):
    import torch
    d = inputs.disk(6000, seed=4)
    _, ref = run_gravity(nc, d, nc.params_default(3, **OVER))
    ctx, a = run_gravity(nc, d, nc.params_default(3, **OVER, p2p_capacity=capacity))
    assert np.array_equal(a, ref)
    del ctx
    # the collision walk, on the same buffer
    far = dict(leaf_size=2, ncs_col=0, ncc_pre_col=0, ncc_post_col=0)
    d = inputs.disk(6000, seed=4)
    d["R"] = d["R"] * 40.0
    want = orc.pairs_brute(d, 1e-2)
    assert len(want) > 0
    ctx, got = run_collide(nc, d, nc.params_default(3, **far, p2p_capacity=capacity), 1e-2)
    assert np.array_equal(got, want)
    del ctx
    torch.cuda.empty_cache()
