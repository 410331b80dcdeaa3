"""A walk beside another stream's long kernels: the waves that find room go on by themselves,
and the results are those of the walk alone, bit for bit."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import dev_arrays, run_collide, run_gravity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def test_walks_beside_a_full_chip(nc):
    import torch
    n, m, dt = 20000, 300000, 0.3
    d, big = inputs.disk(n, seed=41), inputs.disk(m, seed=42)
    prm = nc.params_default(3)
    _, ref = run_gravity(nc, d, prm)
    _, want = run_collide(nc, d, prm, dt)
    # the other stream: sums over every pair, hundreds of workgroups at a time
    other, mine = torch.cuda.Stream(), torch.cuda.Stream()
    hog = nc.Context(nc.params_default(3, gravity_method=nc.GRAVITY_BRUTE_FORCE), m,
                     pair_capacity=1 << 10)
    tb, t = dev_arrays(big), dev_arrays(d)
    ab = [torch.empty(m, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    cap = 1 << 16
    ctx = nc.Context(prm, n, pair_capacity=cap)
    runs = []
    for _ in range(6):
        runs.append(([torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(3)],
                     torch.zeros((cap, 2), dtype=torch.int64, device="cuda:0"),
                     torch.zeros(1, dtype=torch.int64, device="cuda:0")))
    torch.cuda.synchronize()
    hog.build_tree(tb["x"], tb["y"], tb["z"], stream=other)
    for _ in range(3):
        hog.gravity(tb["m"], *ab, stream=other)
    for a, pairs, npairs in runs:
        # the collision walk, then the gravity walk on the same tree
        ctx.build_tree(t["x"], t["y"], t["z"], stream=mine)
        ctx.collide(t["vx"], t["vy"], t["vz"], t["R"], dt, pairs, npairs, stream=mine)
        ctx.gravity(t["m"], *a, stream=mine)
    torch.cuda.synchronize()
    hog.check_status()
    ctx.check_status()
    for a, pairs, npairs in runs:
        assert np.array_equal(torch.stack(a, 1).cpu().numpy(), ref)
        assert np.array_equal(pairs[:int(npairs.item())].cpu().numpy(), want)
