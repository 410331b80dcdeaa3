"""The build's size rules at their edges, against the oracle bit for bit.

The sort forms its boundaries in the counting pass up to 64 buckets (114688 moonlets) and
adds up its counts in the scatter up to 4096 of them (64 buckets of 57 tiles is within,
122880 moonlets beyond); the tree adds up the blocks' counts in the emitting pass up to 128
blocks (131072 moonlets).  Each size is built from a sample, from its own order and after
the moonlets have moved; one bucket and one block with a moonlet more or less are among
them."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.test_gpu_sort import _build, _check_order, _drifted
from tests.test_gpu_tree import nc  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 1023, 1024, 1025, 1792, 1793, 3585, 114688, 114689,
                               122880, 131072, 131073])
def test_builds_at_the_edges(nc, orc, n):  # noqa: F811
    d = inputs.hot_disk(n, seed=31)
    print(f"n {n}", flush=True)
    s = 17
    ctx = nc.Context(nc.params_default(3, leaf_size=s), n, pair_capacity=1 << 16)
    for k, dt in enumerate((0.0, 0.0, 1e-3, 2.0)):
        dk = _drifted(d, dt)
        _build(ctx, dk)
        info = _check_order(ctx, orc, dk, s)
        assert info["sort_prev"] == (1 if k in (1, 2) and n > 1792 else info["sort_prev"])
        t = orc.Tree(dk["x"], dk["y"], dk["z"], s)
        cells = ctx.export("cells")
        for col, want in enumerate((t.level, t.first, t.count, t.child_first, t.nchild,
                                    t.parent)):
            assert np.array_equal(cells[:, col], want), (n, col)
        assert info["nleaves"] == int((t.nchild == 0).sum())
        assert info["maxlevel"] == t.maxlevel
