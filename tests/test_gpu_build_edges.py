"""The build's size rules at their edges, against the oracle bit for bit.

The sort forms its boundaries in the counting pass up to 64 buckets (114688 moonlets) and
adds up its counts in the scatter up to 4096 of them (64 buckets of 57 tiles is within,
122880 moonlets beyond); the tree adds up the blocks' counts in the emitting pass up to 128
blocks (131072 moonlets).  Each size is built from a sample, from its own order and after
the moonlets have moved; one bucket and one block with a moonlet more or less are among
them.  Batched builds sort by (disk, key, index) with the same rules: disks within a bucket
and across many, a bucket of several disks beyond one LDS batch, and plain builds in
between on the same context."""
import numpy as np
import pytest

from paper_2310_20374_amd import inputs
from tests.gpu_util import dev_arrays
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


def _stacked(sizes):
    """Disks with more moonlets on one point than one LDS batch holds."""
    parts = [inputs.hot_disk(k, seed=40 + i) for i, k in enumerate(sizes)]
    for p in parts:
        for c in "xyz":
            p[c][len(p[c]) // 8:] = p[c][0]
    return parts


def _empty():
    return {k: np.zeros(0) for k in inputs.hot_disk(1, seed=0)}


BATCHES = {
    "one_bucket": lambda: [inputs.hot_disk(k, seed=k) if k else _empty()
                           for k in (3, 1, 700, 0, 900)],
    "many_small": lambda: [inputs.hot_disk(1 + k % 23, seed=k) for k in range(400)],
    "mixed": lambda: [inputs.hot_disk(k, seed=k) for k in (20000, 5, 1793, 60000, 50000, 1)],
    "stacked": lambda: _stacked((3000, 9000, 2500, 40)),
}


@pytest.mark.parametrize("case", list(BATCHES))
def test_batched_order(nc, orc, case):  # noqa: F811
    import torch
    parts = BATCHES[case]()
    sizes = [len(p["x"]) for p in parts]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    d = {k: np.concatenate([p[k] for p in parts]) for k in parts[0]}
    n, s = len(d["x"]), 17
    print(f"case {case} n {n}", flush=True)
    ctx = nc.Context(nc.params_default(3, leaf_size=s), n, pair_capacity=1 << 16)
    offd = torch.tensor(off, device="cuda:0")
    for k, dt in enumerate((0.0, 0.0, 1e-3, None, 1e-3, 1.0)):
        if dt is None:                      # a plain build of the same moonlets
            _build(ctx, d)
            _check_order(ctx, orc, d, s)
            continue
        dk = _drifted(d, dt)
        t = dev_arrays(dk)
        ctx.build_tree_batched(offd, t["x"], t["y"], t["z"])
        torch.cuda.synchronize()
        ctx.check_status()
        perm, keys = ctx.export("perm").astype(np.int64), ctx.export("keys")
        for a, b in zip(off[:-1], off[1:]):
            if a == b:
                continue
            o = orc.Tree(*(np.ascontiguousarray(dk[c][a:b]) for c in "xyz"), s)
            assert np.array_equal(perm[a:b], o.perm + a), (k, a)
            assert np.array_equal(keys[a:b], o.keys[o.perm]), (k, a)
