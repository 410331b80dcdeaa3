"""A batch with more leaves than a caller's pair capacity would give direct-sum slots to:
every disk's accelerations are those of the disk alone, bit for bit."""
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


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_batch_equals_alone_with_a_small_pair_capacity(nc, prec):
    import torch
    sizes = (250000, 200001)
    disks = [inputs.disk(n, seed=20 + k) for k, n in enumerate(sizes)]
    # leaves whose sums are split over several waves: some 27 cells of 1000 moonlets each
    prm = nc.params_default(2, leaf_size=16, ncs=1000, ncc_pre=10 ** 6, ncc_post=10 ** 6,
                            walk_waves=256, m2l_capacity=1,
                            precision=nc.FP32_BULK if prec == "fp32" else nc.FP64)
    alone = [run_gravity(nc, d, prm)[1] for d in disks]
    both = {k: np.concatenate([d[k] for d in disks]) for k in disks[0]}
    n = sum(sizes)
    ctx = nc.Context(prm, n, pair_capacity=1 << 14)
    t = dev_arrays(both)
    off = torch.tensor(np.cumsum([0, *sizes]), device="cuda:0")
    a = [torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    ctx.build_tree_batched(off, t["x"], t["y"], t["z"])
    ctx.gravity(t["m"], *a)
    torch.cuda.synchronize()
    ctx.check_status()
    # more leaves than eight slots each fit into the room of 2 (2^17 + 1) words
    assert ctx.tree_info()["nleaves"] > (1 << 15)
    got = torch.stack(a, 1).cpu().numpy()
    assert np.array_equal(got, np.concatenate(alone))
