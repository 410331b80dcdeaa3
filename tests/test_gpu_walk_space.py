"""The space of the walk's hand-down lists: at and beyond what 32-bit offsets reach, and just
enough of it.

A pair list of more than 2^30 entries gives the lists a buffer of more than 2^31 words;
they may use it only up to there.  Whatever the buffer, a walk whose visits fit its
queue_capacity is never refused for the lists' space.  The lists found and the sums over
them are those of the default capacities, bit for bit."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import rel_err, run_collide, run_gravity

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


# Direct-sum pairs of internal cells, which all the leaves below them inherit: far more
# list entries than visits.  (input, leaf size, thresholds, theta)
INHERITED = {
    "disk": (lambda: inputs.disk(6000, seed=7), 1, (512, 512, 2048), 0.4),
    "disk_far": (lambda: inputs.disk(12000, seed=7), 1, (4096, 4096, 16384), 0.4),
    "clumps": (lambda: inputs.clumps(24000, seed=5, n_clumps=8), 4, (512, 512, 2048), 0.4),
    "clumps_small": (lambda: inputs.clumps(12000, seed=5, n_clumps=8), 1, (512, 512, 2048), 0.4),
}


@pytest.mark.parametrize("case", list(INHERITED))
def test_inherited_pairs_need_no_room_of_their_own(nc, orc, case):
    """A walk whose visits and pairs fit the capacities given is not refused for what its
    leaves inherit, and finds the oracle's pairs; the sums are those of the default
    capacities bit for bit."""
    gen, s, thr, theta = INHERITED[case]
    d = gen()
    n = len(d["x"])
    print(f"case {case}", flush=True)
    over = dict(leaf_size=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1], ncc_post=thr[2],
                m2l_per_cell=8192, p2p_per_leaf=8192, walk_waves=256)
    ctx, ref = run_gravity(nc, d, nc.params_default(3, **over))
    i = ctx.tree_info()
    want, _, g = orc.tree_accel(d, p=3, s=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                                ncc_post=thr[2])
    m2l, p2p = g.lists()

    def pairs(v):
        return set(map(tuple, np.sort(np.asarray(v, dtype=np.int64), axis=1).tolist()))

    assert pairs(ctx.export("m2l")) == pairs(m2l) and pairs(ctx.export("p2p")) == pairs(p2p)
    assert rel_err(ref, want)[1] < 1e-11
    # capacities that the visits and the pairs just fit
    tight = dict(queue_capacity=i["visited"], m2l_capacity=1, p2p_capacity=1)
    ctx2 = nc.Context(nc.params_default(3, **over, **tight), n, pair_capacity=1 << 14)
    _, a = run_gravity(nc, d, None, ctx=ctx2)
    assert np.array_equal(a, ref)
    # one visit fewer, and what is asked for then
    tight["queue_capacity"] -= 1
    ctx3 = nc.Context(nc.params_default(3, **over, **tight), n, pair_capacity=1 << 14)
    with pytest.raises(nc.NcorpError) as ei:
        run_gravity(nc, d, None, ctx=ctx3)
    assert ei.value.code == nc.E_CAPACITY and ctx3.get_status()[1] == i["visited"]
