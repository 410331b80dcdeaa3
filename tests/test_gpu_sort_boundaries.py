"""Where the sort's bucket boundaries come from: the last build's order only where the same
context has built as many moonlets before, and only with more than one bucket."""
import pytest

from paper_2310_20374_amd import inputs
from tests.test_gpu_sort import _build, _check_order, _drifted
from tests.test_gpu_tree import nc  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 1024, 1792, 1793, 3585, 114689, 131073])
def test_first_builds_and_single_buckets_take_a_sample(nc, orc, n):  # noqa: F811
    d = inputs.hot_disk(n, seed=31)
    print(f"n {n}", flush=True)
    for fresh in range(2):
        ctx = nc.Context(nc.params_default(3, leaf_size=17), n, pair_capacity=1 << 16)
        for k, dt in enumerate((0.0, 0.0, 1e-3)):
            dk = _drifted(d, dt)
            _build(ctx, dk)
            info = _check_order(ctx, orc, dk, 17)
            assert info["sort_prev"] == (1 if k > 0 and n > 1792 else 0), (fresh, k)
    # another number of moonlets in the same room: no boundaries of its own yet
    if n > 1792:
        other = inputs.hot_disk(n - 1, seed=32)
        _build(ctx, other)
        assert _check_order(ctx, orc, other, 17)["sort_prev"] == 0
