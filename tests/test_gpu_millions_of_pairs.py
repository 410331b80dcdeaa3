"""A collision search that finds more than a million pairs: the ranking's ranges then hold
more keys than LDS.  Two clouds at rest in themselves that meet: every moonlet of one meets
every one of the other within the step, and no other pair can touch."""
import numpy as np
import pytest

from tests.gpu_util import run_collide
from tests.test_gpu_resolve import FIELDS, _gpu_steps, _per_step

pytestmark = pytest.mark.gpu
DT = 0.5


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def _clouds(a, b):
    rng = np.random.default_rng(a)
    x = 0.01 * rng.random((a + b, 3)) + 1.0
    x[a:, 0] += 1.0
    v = np.zeros_like(x)
    v[:a, 0], v[a:, 0] = 1.0, -1.0
    d = {c: np.ascontiguousarray(x[:, i]) for i, c in enumerate("xyz")}
    d.update({"v" + c: np.ascontiguousarray(v[:, i]) for i, c in enumerate("xyz")})
    d["m"], d["R"] = np.full(a + b, 1e-6), np.full(a + b, 0.2)
    want = np.stack(np.meshgrid(np.arange(a), np.arange(a, a + b), indexing="ij"), -1)
    return d, want.reshape(-1, 2)


# 1.3 million pairs: few ranges beyond 4096 keys; 4 million: nearly all of them
@pytest.mark.parametrize("a,b", [(1150, 1151), (2000, 2003)])
def test_millions_of_pairs(nc, a, b):
    d, want = _clouds(a, b)
    print(f"{len(want)} pairs", flush=True)
    _, got = run_collide(nc, d, nc.params_default(3, leaf_size=64), DT, cap=1 << 22)
    assert np.array_equal(got, want)


def test_millions_of_pairs_resolved(nc, orc):
    d, want = _clouds(1150, 1151)
    prm = nc.params_default(0, M_central=0.0, leaf_size=64,
                            collision_mode=nc.COLLISIONS_RESOLVE, collision_f=1.5)
    got, pairs, cnt = _gpu_steps(nc, d, prm, DT, 1, cap=1 << 21)
    ref, rp = orc.kdk_steps(d, DT, 1, None, M_central=0.0,
                            collide_fn=lambda q, h: want, resolve_f=1.5)
    assert np.array_equal(_per_step(pairs, cnt)[0], rp[0])
    for k in FIELDS:
        assert np.array_equal(got[k], ref[k]), k
