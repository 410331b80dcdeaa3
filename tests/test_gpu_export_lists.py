"""The pair lists that ncorp_export_host gives back: empty where the last walk wrote none
(nothing is read by the indices of an earlier one), and the same pairs as counted."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import dev_arrays, run_gravity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def test_no_lists_after_a_walk_that_did_not_run(nc):
    import torch
    n = 30000
    d = inputs.disk(n, seed=2)
    ctx, _ = run_gravity(nc, d, nc.params_default(3, leaf_size=4))
    assert len(ctx.export("p2p")) > 0 and len(ctx.export("m2l")) > 0
    t = dev_arrays(d)
    a = [torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    # offsets that don't end at n: every pass of the call does nothing
    off = torch.tensor([0, 10, n - 1], dtype=torch.int64, device="cuda:0")
    ctx.build_tree_batched(off, t["x"], t["y"], t["z"])
    ctx.gravity(t["m"], *a)
    torch.cuda.synchronize()
    assert ctx.get_status()[0] == nc.E_INVALID
    assert len(ctx.export("p2p")) == 0 and len(ctx.export("m2l")) == 0
    # and the next call's lists are its own again
    run_gravity(nc, d, None, ctx=ctx)
    info = ctx.tree_info()
    assert len(ctx.export("p2p")) == info["p2p"] and len(ctx.export("m2l")) == info["m2l"]


@pytest.mark.parametrize("n,s", [(300, 300), (5000, 1), (200000, 17)])
def test_every_pair_is_given_back_once(nc, n, s):
    d = inputs.disk(n, seed=3)
    ctx, _ = run_gravity(nc, d, nc.params_default(3, leaf_size=s, ncs=64, ncc_pre=64,
                                                  ncc_post=256))
    info = ctx.tree_info()
    for what in ("m2l", "p2p"):
        v = np.sort(ctx.export(what).astype(np.int64), axis=1)
        assert len(v) == info[what]
        assert len(np.unique(v[:, 0] << 32 | v[:, 1])) == len(v)
