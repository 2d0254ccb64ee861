"""A thread's tuning is the pair that cxbwt_get_tuning reads and nothing else:
setting it again restores the thread, and the default pair leaves the choice to
the library at every size."""
import ctypes

import pytest

from paper_1401_7457_amd import autotune, cxbwt

SIZES = (1, 1_000_000, 11_999_999, 12_000_000, 16_000_000, 4_000_000_000)


def test_saved_and_set_again_is_what_it_was():
    unchosen = [cxbwt.build_tuning(n) for n in SIZES]
    assert unchosen[0] == cxbwt.TUNING_CHOICES[0] and unchosen[-1] == (16, 8)
    before = cxbwt.get_tuning()
    for choice in cxbwt.TUNING_CHOICES[1:]:
        cxbwt.set_tuning(*choice)
        try:
            assert all(cxbwt.build_tuning(n) == choice for n in SIZES)  # a choice holds at every size
        finally:
            cxbwt.set_tuning(*before)
        assert [cxbwt.build_tuning(n) for n in SIZES] == unchosen
    held = autotune.current()
    autotune.apply((16, 6, cxbwt.SCHEDULE_STRINGWORD))
    autotune.apply(held)
    assert [cxbwt.build_tuning(n) for n in SIZES] == unchosen and cxbwt.get_schedule() == cxbwt.SCHEDULE_MSD


def test_null_pointers_are_refused():
    v = ctypes.c_uint32()
    L = cxbwt.lib()
    assert L.cxbwt_build_tuning(10, 1, None, ctypes.byref(v)) == cxbwt.EINVAL
    assert L.cxbwt_build_tuning(10, 1, ctypes.byref(v), None) == cxbwt.EINVAL
    assert L.cxbwt_build_tuning(10, 0, ctypes.byref(v), ctypes.byref(v)) == cxbwt.EINVAL


@pytest.mark.parametrize("mean,tile", [(500, 8), (2048, 8), (2049, 16), (100_000, 16)])
def test_collections_below_a_tile_keep_the_narrow_one(mean, tile):
    for count in (10_000, 100_000):
        got = cxbwt.build_tuning(mean * count, count)
        assert got == ((tile, 8) if mean * count >= 12_000_000 else cxbwt.TUNING_CHOICES[0])


@pytest.mark.parametrize("ms,best", [({(8, 6): 1.01, (16, 8): 1.0, (8, 3): 1.4}, (8, 6)),
                                     ({(8, 6): 1.05, (16, 8): 1.0, (8, 3): 1.4}, (16, 8)),
                                     ({(16, 8): 1.0, (8, 3): 0.9}, (8, 3))])
def test_tuner_takes_the_default_of_equal_choices(ms, best):
    # the default, not the pair it stands for at this size: the remembered
    # choice is applied to other sizes of the class
    assert autotune.fastest({(*k, cxbwt.SCHEDULE_MSD): v for k, v in ms.items()}) == (*best, cxbwt.SCHEDULE_MSD)
