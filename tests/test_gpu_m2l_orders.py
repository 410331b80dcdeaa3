"""Interaction tensors of every order and precision, over lists of one batch of 64 sources
and of several, against the oracle tree.  In FP64 the sums differ in order only (1e-11); in
FP32 offsets and bulk arithmetic are rounded (rms 1e-6, closest pairs 1e-4, the bounds of
every FP32 comparison with leaves much smaller than the disk)."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import rel_err, run_gravity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


@pytest.mark.parametrize("theta", [0.7, 0.3])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
def test_every_order(nc, orc, p, prec, theta):
    d = inputs.disk(6000, seed=51)
    s, thr = 8, (64, 8, 64)
    print(f"p {p} {prec} theta {theta}", flush=True)
    prm = nc.params_default(p, leaf_size=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                            ncc_post=thr[2],
                            precision=nc.FP32_BULK if prec == "fp32" else nc.FP64)
    ctx, a = run_gravity(nc, d, prm)
    ref, _, g = orc.tree_accel(d, p=p, s=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                               ncc_post=thr[2])
    m2l, _ = g.lists()
    longest = np.bincount(np.asarray(m2l).reshape(-1)).max()
    rms, mx = rel_err(a, ref)
    print(f"  longest list {longest}, rms {rms:.3e} max {mx:.3e}", flush=True)
    if prec == "fp64":
        assert mx < 1e-11
    else:
        assert rms <= 1e-6 and mx <= 1e-4
    _, b = run_gravity(nc, d, None, ctx=ctx)
    assert rel_err(b, a)[1] < 1e-11
