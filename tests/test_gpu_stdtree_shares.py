"""The standard tree code with one, two and four lanes a moonlet, at the sizes where the
number changes, against the oracle (FP64 sums in another order: 1e-11).  A batch of disks
large enough for one lane a moonlet gives the sums of each disk alone, with four, bit for
bit."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import dev_arrays, rel_err, run_gravity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def _prm(nc, p):
    return nc.params_default(p, leaf_size=102, gravity_method=nc.GRAVITY_STANDARD_TREE,
                             ncb_pre=6, ncb_post=16)


@pytest.mark.parametrize("n,p", [(15, 3), (17, 6), (33, 3), (40001, 4), (65536, 3),
                                 (65537, 3)])
def test_shares_match_oracle(nc, orc, n, p):
    d = inputs.hot_disk(n, seed=61)
    print(f"n {n} p {p}", flush=True)
    _, a = run_gravity(nc, d, _prm(nc, p))
    ref, _, _ = orc.standard_tree_accel(d, p=p, s=102, ncb_pre=6, ncb_post=16)
    assert rel_err(a, ref)[1] < 1e-11


def test_batch_equals_each_disk(nc):
    import torch
    parts = [inputs.hot_disk(k, seed=k) for k in (70000, 3, 1500, 40001)]
    off = np.concatenate([[0], np.cumsum([len(p["x"]) for p in parts])]).astype(np.int64)
    d = {k: np.concatenate([p[k] for p in parts]) for k in parts[0]}
    n = len(d["x"])
    ctx = nc.Context(_prm(nc, 3), n, pair_capacity=1 << 10)
    t = dev_arrays(d)
    a = [torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    ctx.build_tree_batched(torch.tensor(off, device="cuda:0"), t["x"], t["y"], t["z"])
    ctx.gravity(t["m"], *a)
    torch.cuda.synchronize()
    ctx.check_status()
    a = torch.stack(a, 1).cpu().numpy()
    for k, part in enumerate(parts):
        _, one = run_gravity(nc, part, _prm(nc, 3))
        assert np.array_equal(a[off[k]:off[k + 1]], one), k
