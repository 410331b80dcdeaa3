"""The largest systems that the allocation-free form's declaration names."""
import pytest

from paper_2310_20374_amd import ncorp


@pytest.mark.parametrize("p,leaf,largest", [(6, 52, 18810), (4, 52, 19824), (3, 17, 7048)])
def test_largest_system_without_a_workspace(p, leaf, largest):
    prm = ncorp.params_default(p, leaf_size=leaf)
    limit = ncorp.STATIC_WORKSPACE_BYTES
    assert ncorp.workspace_bytes(prm, largest, 1) <= limit
    assert ncorp.workspace_bytes(prm, largest + 1, 1) > limit
