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


@pytest.mark.parametrize("disks", [1, 3, 600])
def test_radix_sort_of_large_builds(nc, orc, disks):  # noqa: F811
    """More moonlets than the bucket sort takes (3200 buckets): the radix sort's order."""
    import torch
    n = 3200 * 1792 + 4097
    g = torch.Generator(device="cuda:0").manual_seed(7)
    x, y, z = (torch.randn(n, generator=g, device="cuda:0", dtype=torch.float64).clamp_(-2, 2)
               for _ in range(3))
    x[100:300] = x[100]                                 # equal keys keep their order
    y[100:300] = y[100]
    z[100:300] = z[100]
    print(f"n {n} disks {disks}", flush=True)
    ctx = nc.Context(nc.params_default(0, leaf_size=64), n, pair_capacity=1 << 12)
    off = torch.linspace(0, n, disks + 1).round().to(torch.int64)
    off[-1] = n
    if disks == 1:
        ctx.build_tree(x, y, z)
    else:
        ctx.build_tree_batched(off.to("cuda:0"), x, y, z)
    torch.cuda.synchronize()
    ctx.check_status()
    keys = ctx.export("keys")
    perm = ctx.export("perm").astype(np.int64)
    assert np.array_equal(np.sort(perm), np.arange(n))
    o = off.numpy()
    inner = np.ones(n - 1, bool)
    inner[o[1:-1] - 1] = False                          # across a disk boundary
    up = (keys[1:] > keys[:-1]) | ((keys[1:] == keys[:-1]) & (perm[1:] > perm[:-1]))
    assert up[inner].all()
    assert np.array_equal(np.searchsorted(o, perm, side="right"),
                          np.searchsorted(o, np.arange(n), side="right"))
    # the keys themselves, on a sample of one disk against the oracle
    if disks == 1:
        L = float(ctx.tree_info()["L"]) if "L" in ctx.tree_info() else 2.0 ** 2
        take = np.sort(np.random.default_rng(1).choice(n, 4000, replace=False))
        xs = [v.cpu().numpy()[perm[take]] for v in (x, y, z)]
        t = orc.Tree(*(np.ascontiguousarray(v) for v in xs), 8, L)
        assert np.array_equal(t.keys, keys[take])
