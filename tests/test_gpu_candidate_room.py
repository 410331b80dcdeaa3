"""Collision candidates beyond the room of p2p_capacity pairs: the call is refused, and the
size it asks for is one that suffices, however far the list was outgrown."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import dev_arrays

pytestmark = pytest.mark.gpu
DT = 1e-3


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def _search(nc, d, prm, lists):
    """The pairs of d, and the context: after the collision walk, or on the lists of a
    gravity evaluation."""
    import torch
    n, cap = len(d["x"]), 1 << 18
    ctx = nc.Context(prm, n, pair_capacity=cap)
    t = dev_arrays(d)
    pairs = torch.zeros((cap, 2), dtype=torch.int64, device="cuda:0")
    npairs = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    ctx.build_tree(t["x"], t["y"], t["z"])
    if lists:
        ctx.gravity(t["m"], *[torch.empty(n, dtype=torch.float64, device="cuda:0")
                              for _ in range(3)])
    ctx.collide(t["vx"], t["vy"], t["vz"], t["R"], DT, pairs, npairs)
    torch.cuda.synchronize()
    return ctx, pairs, npairs


@pytest.mark.parametrize("lists", [False, True])
def test_required_room_suffices(nc, orc, lists):
    # leaves of a few moonlets whose spheres reach many neighbouring leaves
    d = inputs.disk(20000, seed=9)
    d["R"] = np.full_like(d["R"], 0.35)
    over = dict(leaf_size=4, walk_waves=256, ncs_col=0, ncc_pre_col=0, ncc_post_col=0)
    full, pairs, npairs = _search(nc, d, nc.params_default(3, **over), lists)
    full.check_status()
    count = full.tree_info()["col_cand"]
    # more than twice what p2p_capacity = 1 (and 2^17 on top) holds
    assert count > 2 * (1 << 17) + (1 << 14), count
    k = int(npairs.item())
    want = pairs[:min(k, pairs.shape[0])].cpu().numpy()
    small, _, _ = _search(nc, d, nc.params_default(3, **over, p2p_capacity=1), lists)
    status, required, _ = small.get_status()
    assert status == nc.E_CAPACITY and required >= count
    again, pairs, npairs = _search(nc, d, nc.params_default(3, **over, p2p_capacity=required),
                                   lists)
    again.check_status()
    assert int(npairs.item()) == k and again.tree_info()["col_cand"] == count
    assert np.array_equal(pairs[:len(want)].cpu().numpy(), want)
