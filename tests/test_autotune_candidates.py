"""What the autotuner measures by default: the library's own launch shape among the others,
and only shapes that the library takes."""
import ctypes as C

from paper_2310_20374_amd import autotune, ncorp


def test_defaults_are_among_the_candidates():
    prm = ncorp.params_default(6)
    assert prm.walk_waves in autotune.WALK_WAVES
    # 0 stands for a tile of 256 and 4 targets
    assert (prm.p2p_tile or 256, prm.p2p_targets_max or 4) in autotune.TILE_SHAPES


def test_candidates_are_accepted():
    shapes = [dict(leaf_size=s) for s in autotune.CANDIDATES]
    shapes += [dict(p2p_tile=t, p2p_targets_max=m) for t, m in autotune.TILE_SHAPES]
    shapes += [dict(walk_waves=w) for w in autotune.WALK_WAVES]
    for over in shapes:
        h = C.c_void_p()
        prm = ncorp.params_default(4, **over)
        assert ncorp.lib().ncorp_create(C.byref(prm), C.byref(h)) == ncorp.OK, over
        ncorp.lib().ncorp_destroy(h)
