"""Neighbourhood scans by rows of the dense grid, where a row or a plane is missing.

With the dense grid the three cells along x of each of the nine rows are one run of the
sorted moonlets.  The inputs: a single plane, single rows along each axis, two crowded
cells at the box's ends, a box with many empty cells; and a step, whose build brings the
masses along, against a kick from a separate evaluation.  Bounds as for every mesh case:
sums of the same pairs, in FP64 (1e-11); pairs and counts equal."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import rel_err
from tests.test_gpu_mesh import _gpu_steps, _mesh_run, _prm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nc():
    from paper_2310_20374_amd import ncorp
    ncorp.lib()
    return ncorp


def _gas(n, flat="", scale=1.0):
    d = inputs.gas_box(n, seed=21, radius=2e-3)
    for k in "xyz":
        d[k] = d[k] * scale
    for k in flat:
        d[k] = np.zeros(n)
    return d


def _crowded(n):
    d = _gas(n)
    half = np.arange(n) < n // 2
    for k in "xyz":
        d[k] = 0.04 * (d[k] - d[k].min()) / (d[k].max() - d[k].min()) + 0.005
        d[k][half] += 1.0
    return d


CASES = {
    # name: (input, gamma)
    "plane": (lambda: _gas(3000, "z"), 0.05),
    "row_x": (lambda: _gas(2000, "yz"), 0.01),
    "row_y": (lambda: _gas(2000, "xz"), 0.01),
    "row_z": (lambda: _gas(2000, "xy"), 0.01),
    "crowded": (lambda: _crowded(601), 0.05),
    "mostly_empty": (lambda: _gas(1500, "", 1.0), 0.03),
}


@pytest.mark.parametrize("case", list(CASES))
def test_rows_match_oracle(nc, orc, case):
    gen, g = CASES[case]
    d, dt = gen(), 0.004
    print(f"case {case}", flush=True)
    a, pairs, st, _ = _mesh_run(nc, d, _prm(nc, g, 64), dt)
    assert rel_err(a, orc.mesh_accel(d, g))[1] < 1e-11
    assert np.array_equal(pairs, orc.mesh_pairs(d, g, dt))
    assert st["neighbours"] == orc.mesh_neighbours(d, g)


def test_step_brings_the_masses_along(nc):
    """A step's first half kick, seen in its first drift, is that of the accelerations of
    build_mesh and gravity: positions after one step equal x + dt (v + dt/2 a) to rounding."""
    d, g, dt = _gas(3000), 0.05, 1e-3
    d["R"][:5] = 0.1                                   # out of the mesh
    prm = _prm(nc, g, 64, M_central=0.0)
    a, _, _, _ = _mesh_run(nc, d, prm, dt)
    got, _, _, _ = _gpu_steps(nc, d, prm, dt, 1)
    for k, c in enumerate("xyz"):
        want = d[c] + dt * (d["v" + c] + 0.5 * dt * a[:, k])
        assert np.abs(got[c] - want).max() < 1e-14 * np.abs(d[c]).max()


@pytest.mark.parametrize("n", [4096, 4097, 65536, 65537])
def test_sort_at_its_edges(nc, orc, n):
    """The mesh's sort at the edges of a tile and of its groups of tiles.  A massless
    moonlet far away makes the box larger than the dense grid, so that the cells are
    hashed and sorted by all digits: the same sums and pairs in another order."""
    d = _gas(n)
    g, dt = (n ** (-1 / 3)) * 1.3, 1e-4
    d["R"][:] = 0.2 * g
    d["R"][1] = 2 * g                                   # out of the mesh
    d["m"][0], d["R"][0] = 0.0, 1e-9
    far = {k: v.copy() for k, v in d.items()}
    for k in "xyz":
        d[k][0], far[k][0] = 1.2, 40.0
    print(f"n {n}", flush=True)
    a, pairs, st, _ = _mesh_run(nc, d, _prm(nc, g, 64), dt, cap=1 << 18)
    b, fpairs, fst, _ = _mesh_run(nc, far, _prm(nc, g, 64), dt, cap=1 << 18)
    assert st["n_out"] == 1 and fst["n_out"] == 1
    assert rel_err(a[1:], b[1:])[1] < 1e-11
    assert np.array_equal(pairs, fpairs)
    assert np.array_equal(pairs, orc.pairs_grid(d, dt))
    if n <= 4097:
        assert rel_err(a[1:], orc.mesh_accel(d, g)[1:])[1] < 1e-11
        assert st["neighbours"] == orc.mesh_neighbours(d, g)
