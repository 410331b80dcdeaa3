"""Collision searches that find many pairs: lists ranked by counting all against all (up to
4096 pairs) and by ranges (beyond), waves that find more pairs than they hold back, and
matchings whose first round is spread over several blocks (more than 4096 pairs).  The
pairs are the oracle's, in order; without gravity the resolved states agree bit for bit."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import run_collide
from tests.test_gpu_resolve import FIELDS, _gpu_steps, _per_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def _head_on(m):
    """m pairs (k, k + m), far from each other, that meet within the step."""
    k = np.arange(m)
    side = int(np.ceil(m ** (1 / 3)))
    base = np.stack([k % side, k // side % side, k // side ** 2], 1) / side + 1.0   # none at the origin
    x = np.concatenate([base, base + [0.1 / side, 0, 0]])
    v = np.zeros_like(x)
    v[:m, 0] = 0.1 / side
    d = {c: np.ascontiguousarray(x[:, i]) for i, c in enumerate("xyz")}
    d.update({"v" + c: np.ascontiguousarray(v[:, i]) for i, c in enumerate("xyz")})
    rng = np.random.default_rng(3)
    d["m"], d["R"] = np.full(2 * m, 1e-6), np.full(2 * m, 0.02 / side)
    p = rng.permutation(2 * m)
    return {c: np.ascontiguousarray(a[p]) for c, a in d.items()}


def _star(n):
    """One moonlet that every other one meets, all pairs with the same smaller index: the
    others on a sphere around it, moving inwards."""
    rng = np.random.default_rng(5)
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    u[0] = 0.0
    x, v = 0.5 * u + 2.0, -u               # none at the origin
    d = {c: np.ascontiguousarray(x[:, i]) for i, c in enumerate("xyz")}
    d.update({"v" + c: np.ascontiguousarray(v[:, i]) for i, c in enumerate("xyz")})
    d["m"], d["R"] = np.full(n, 1e-6), np.full(n, 1e-6)
    d["R"][0] = 0.4999
    return d


CASES = {
    # name: (input, dt, leaf size)
    "head_on_4096": (lambda: _head_on(4096), 1.0, 8),
    "head_on_4097": (lambda: _head_on(4097), 1.0, 8),
    "gas_overlapping": (lambda: inputs.gas_box(3000, seed=7, radius=0.03), 0.06, 8),
    "gas_crowded": (lambda: inputs.gas_box(1500, seed=8, radius=0.15), 0.1, 128),
    "star": (lambda: _star(6000), 1e-3, 16),
}


@pytest.mark.parametrize("case", list(CASES))
def test_many_pairs(nc, orc, case):
    gen, dt, s = CASES[case]
    d = gen()
    want = orc.pairs_brute(d, dt)
    print(f"case {case}: {len(want)} pairs", flush=True)
    assert len(want) >= 4096
    prm = nc.params_default(3, leaf_size=s)
    _, got = run_collide(nc, d, prm, dt, cap=1 << 20)
    assert np.array_equal(got, want)
    # a step: the search on the gravity walk's lists is the tree's own without gravity
    for mode in (nc.COLLISIONS_REPORT, nc.COLLISIONS_RESOLVE):
        prm = nc.params_default(0, M_central=0.0, leaf_size=s, collision_mode=mode,
                                collision_f=1.5)
        got, pairs, cnt = _gpu_steps(nc, d, prm, dt, 1, cap=1 << 20)
        ref, rp = orc.kdk_steps(d, dt, 1, None, M_central=0.0,
                                collide_fn=lambda q, h: orc.pairs_brute(q, h),
                                resolve_f=1.5 if mode == nc.COLLISIONS_RESOLVE else None)
        assert np.array_equal(_per_step(pairs, cnt)[0], rp[0])
        for k in FIELDS:
            assert np.array_equal(got[k], ref[k]), k


def test_many_pairs_on_the_gravity_lists(nc, orc):
    d = inputs.gas_box(4000, seed=9, radius=0.03)
    d["m"][:] = 1e-12
    dt = 0.04
    prm = nc.params_default(3, M_central=0.0, leaf_size=16)
    _, pairs, cnt = _gpu_steps(nc, d, prm, dt, 1, cap=1 << 20)
    a, _, _ = orc.tree_accel(d, p=3, s=16)
    v = {c: d["v" + c] + 0.5 * dt * a[:, k] for k, c in enumerate("xyz")}
    moved = dict(d, **{"v" + c: v[c] for c in "xyz"})
    want = orc.pairs_brute(moved, dt)
    print(f"{len(want)} pairs", flush=True)
    assert len(want) > 4096 and np.array_equal(pairs[:, 1:], want)
