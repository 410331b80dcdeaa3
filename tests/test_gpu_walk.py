"""The gravity walk's capacities and its hand-down lists at their edges.

A walk takes the space of its hand-down lists from the room of queue_capacity visits, or
from that of the direct-sum pair list where the caller's queue is smaller than that list
(then without the per-cell slots), and spills lists beyond a cell's slot, or beyond the
256 entries a wave stages, into linked segments.  None of this may change a list: the
cell-pair sets stay the oracle's, and the accelerations those of the default capacities
bit for bit.  A walk that visits more pairs than queue_capacity, or finds more pairs than
a pair list holds, is refused with the size that would have fitted."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import run_gravity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


# (input, p, leaf size, thresholds, theta): default lists; long hand-down lists (small
# opening angle, small leaves); direct-sum pairs of internal cells, which the leaves
# below inherit (thresholds far above the leaf size); one chain of single children
CASES = {
    "disk": (lambda: inputs.disk(20000, seed=3), 4, 24, (64, 8, 64), 0.5),
    "long": (lambda: inputs.disk(6000, seed=4), 3, 2, (0, 0, 0), 0.25),
    "inherited": (lambda: inputs.clumps(8000, seed=5, n_clumps=8), 3, 4, (512, 512, 2048), 0.4),
    "stacked": (lambda: inputs.coincident(500, seed=6), 3, 8, (64, 8, 64), 0.5),
}


def _params(nc, case, **over):
    _, p, s, thr, theta = CASES[case]
    return nc.params_default(p, leaf_size=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                             ncc_post=thr[2], m2l_per_cell=8192, p2p_per_leaf=8192, **over)


@pytest.mark.parametrize("case", list(CASES))
def test_lists_and_space_at_their_edges(nc, orc, case):
    gen, p, s, thr, theta = CASES[case]
    d = gen()
    print(f"case {case}", flush=True)
    ctx, a = run_gravity(nc, d, _params(nc, case))
    info = ctx.tree_info()
    _, _, g = orc.tree_accel(d, p=p, s=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                             ncc_post=thr[2])
    m2l, p2p = g.lists()

    def pairs(v):
        return set(map(tuple, np.sort(np.asarray(v, dtype=np.int64), axis=1).tolist()))

    assert pairs(ctx.export("m2l")) == pairs(m2l) and pairs(ctx.export("p2p")) == pairs(p2p)
    assert info["m2l"] == len(m2l) and info["p2p"] == len(p2p)
    # exactly enough room for the visits: the same lists from the other space
    _, b = run_gravity(nc, d, _params(nc, case, queue_capacity=info["visited"]))
    assert np.array_equal(a, b)
    # fewer workgroups than cells: the same again
    _, b = run_gravity(nc, d, _params(nc, case, walk_waves=256))
    assert np.array_equal(a, b)


@pytest.mark.parametrize("field,n", [("queue_capacity", 40000), ("m2l_capacity", 40000),
                                     ("p2p_capacity", 40000), ("p2p_capacity", 120000)])
def test_walk_beyond_its_capacity_is_refused(nc, field, n):
    # the pair counts get 2^17 on top of the value given with 256 or 512 walk waves
    d = inputs.disk(n, seed=7)
    over = dict(leaf_size=2, ncs=0, ncc_pre=0, ncc_post=0, walk_waves=256)
    full, ref = run_gravity(nc, d, nc.params_default(3, **over))
    info = full.tree_info()
    count = {"queue_capacity": info["visited"], "m2l_capacity": info["m2l"] - (1 << 17),
             "p2p_capacity": info["p2p"] - (1 << 17)}[field]
    del full
    ctx = nc.Context(nc.params_default(3, **over, **{field: 1}), n, pair_capacity=1 << 14)
    if count <= 1:
        _, a = run_gravity(nc, d, None, ctx=ctx)
        assert np.array_equal(a, ref)
        return
    with pytest.raises(nc.NcorpError) as ei:
        run_gravity(nc, d, None, ctx=ctx)
    assert ei.value.code == nc.E_CAPACITY
    req = ctx.get_status()[1]
    assert req > 1
    _, a = run_gravity(nc, d, nc.params_default(3, **over, **{field: int(req)}))
    assert np.array_equal(a, ref)
