"""Direct sums dealt to several waves a leaf, at the edges of the deal.

A leaf's sums are split into up to eight slots by the work it has, its list taken 64
source cells and 256 moonlets at a time; FP32 deals strands of whole batches of cells (one
strand up to 64 cells, eight beyond), FP64 equal shares.  The cases: a tree of one leaf below, at and above a wave and a tile; few leaves of several
target chunks; lists beyond 64 cells with fewer and with more batches than slots; a tree
with and one without split leaves; a tile of 128 and of 512.  FP64 differs from the
oracle by the order of sums only (1e-11).  In FP32 an offset from the leaf centre carries
6e-8 of the leaf size: up to 6000 moonlets, whose leaves may be as large as the disk, are
held to that rounding pair by pair, more to the bounds of the oracle comparisons with
leaves much smaller than the disk (rms 1e-6, closest pairs 1e-4)."""
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


NONE, ALL, USUAL = (0, 0, 0), (10 ** 9, 8, 64), (64, 8, 64)
CASES = {
    # name: (N, leaf size, thresholds, theta, tile)
    "one_leaf_5": (5, 8, USUAL, 0.5, 0),
    "one_leaf_64": (64, 64, USUAL, 0.5, 0),
    "one_leaf_65": (65, 128, USUAL, 0.5, 0),
    "one_leaf_257": (257, 512, USUAL, 0.5, 0),
    "one_leaf_1024": (1024, 1024, USUAL, 0.5, 0),
    "few_leaves_of_chunks": (3000, 512, USUAL, 0.5, 0),
    "lists_of_many_batches": (3000, 2, ALL, 0.5, 0),
    "lists_of_few_batches": (2000, 16, ALL, 0.5, 0),
    "long_lists": (6000, 2, NONE, 0.25, 0),
    "split": (20000, 24, USUAL, 0.5, 0),
    "split_tile_128": (9000, 24, USUAL, 0.5, 128),
    "split_tile_512": (9000, 24, USUAL, 0.5, 512),
    "unsplit": (60000, 4, NONE, 0.7, 0),
}


def offset_rounding(d):
    """Bound on the FP32 error of every moonlet's sum: with u = 2^-24, an offset o from the
    centre is rounded by u |o|, a separation by u (|o_i| + |o_j| + r) in each of three
    components, a term m/r^2 by four times that over r and by further roundings, some eight
    in a direct sum and 64 in an expansion; the centre is within the moonlets' box."""
    x = np.stack([d["x"], d["y"], d["z"]], 1)
    size = np.linalg.norm(x.max(0) - x.min(0))       # >= |o|
    r = np.linalg.norm(x[:, None] - x[None], axis=2)
    np.fill_diagonal(r, np.inf)
    term = d["m"][None] / r ** 2
    per = np.where(np.isfinite(r), 4 * np.sqrt(3) * (2 * size / r + 1) + 64, 0)
    return 2.0 ** -24 * (term * per).sum(1)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", list(CASES))
def test_split_sums_match_oracle(nc, orc, case, prec):
    n, s, thr, theta, tile = CASES[case]
    d = inputs.disk(n, seed=11)
    print(f"case {case} {prec}", flush=True)
    prm = nc.params_default(3, leaf_size=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                            ncc_post=thr[2], p2p_tile=tile, m2l_per_cell=8192,
                            p2p_per_leaf=8192,
                            precision=nc.FP32_BULK if prec == "fp32" else nc.FP64)
    ctx, a = run_gravity(nc, d, prm)
    ref, _, _ = orc.tree_accel(d, p=3, s=s, theta_min=theta, ncs=thr[0], ncc_pre=thr[1],
                               ncc_post=thr[2])
    rms, mx = rel_err(a, ref)
    print(f"  rms {rms:.3e} max {mx:.3e}", flush=True)
    if prec == "fp64":
        assert mx < 1e-11
    elif n <= 6000:
        assert np.all(np.linalg.norm(a - ref, axis=1) <= offset_rounding(d))
    else:
        assert rms <= 1e-6 and mx <= 1e-4
    # the same sums again: the waves' parts are added in a fixed order
    _, b = run_gravity(nc, d, None, ctx=ctx)
    if prec == "fp32":
        assert np.array_equal(a, b)
    else:
        assert rel_err(b, a)[1] < 1e-11


def test_more_leaves_than_room_for_slots(nc):
    """A pair list with less room than there are leaves holds no slots either: every leaf
    is then one wave's, with the sums that the default room gives."""
    d = inputs.disk(300000, seed=12)
    over = dict(leaf_size=1, ncs=65536, ncc_pre=65536, ncc_post=65536, walk_waves=256)
    _, a = run_gravity(nc, d, nc.params_default(2, **over))
    _, b = run_gravity(nc, d, nc.params_default(2, m2l_capacity=1, **over))
    assert rel_err(b, a)[1] < 1e-11
