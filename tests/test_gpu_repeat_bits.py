"""The same call on the same input gives the same bits, on the same context and on another:
every floating-point sum has an order of its own, however its work was dealt out."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import run_gravity
from tests.test_gpu_direct_split import CASES
from tests.test_gpu_resolve import FIELDS, _gpu_steps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def _three_times(nc, d, prm):
    ctx, a = run_gravity(nc, d, prm)
    _, b = run_gravity(nc, d, None, ctx=ctx)
    _, c = run_gravity(nc, d, prm)
    assert np.array_equal(a, b) and np.array_equal(a, c)


def _prec(nc, prec):
    return nc.FP32_BULK if prec == "fp32" else nc.FP64


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", list(CASES))
def test_direct_sums(nc, case, prec):
    n, s, thr, theta, tile = CASES[case]
    _three_times(nc, inputs.disk(n, seed=11),
                 nc.params_default(3, leaf_size=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                                   ncc_post=thr[2], p2p_tile=tile, m2l_per_cell=8192,
                                   p2p_per_leaf=8192, precision=_prec(nc, prec)))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
def test_interaction_tensors(nc, p, prec):
    _three_times(nc, inputs.disk(6000, seed=51),
                 nc.params_default(p, leaf_size=8, theta_min=0.3, ncs=64, ncc_pre=8, ncc_post=64,
                                   precision=_prec(nc, prec)))


@pytest.mark.parametrize("n", [700, 9973, 200001])
@pytest.mark.parametrize("method", ["falcon", "standard", "brute"])
def test_methods(nc, method, n):
    if method == "brute" and n > 10000:
        pytest.skip("O(n^2)")
    g = {"falcon": nc.GRAVITY_FALCON, "standard": nc.GRAVITY_STANDARD_TREE,
         "brute": nc.GRAVITY_BRUTE_FORCE}[method]
    _three_times(nc, inputs.hot_disk(n, seed=5), nc.params_default(6, gravity_method=g))


@pytest.mark.parametrize("method", ["falcon", "mesh"])
def test_steps(nc, method):
    over = dict(collision_mode=nc.COLLISIONS_RESOLVE)
    if method == "mesh":
        over.update(gravity_method=nc.GRAVITY_MESH, collision_method=nc.COLLISIONS_MESH)
    # (the clumps' mesh would be finer than many of its moonlets)
    d = inputs.disk(30000, seed=6) if method == "mesh" else inputs.clumps(30000, seed=6,
                                                                          n_clumps=20)
    runs = [_gpu_steps(nc, d, nc.params_default(4, **over), 1e-3, 3) for _ in range(2)]
    (a, pa, ca), (b, pb, cb) = runs
    assert np.array_equal(ca, cb) and np.array_equal(pa, pb)
    for k in FIELDS:
        assert np.array_equal(a[k], b[k]), k
