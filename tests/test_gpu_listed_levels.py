"""Builds whose levels are listed fit the scratch of one batch at every size
from which level 1 leaves segments: the device finishes them, without a level
left to the host."""
import sys

import numpy as np
import pytest

from oracle import oracle
from paper_1401_7457_amd import cxbwt, datagen

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    cxbwt.lib()
    before = cxbwt.get_tuning()
    yield
    cxbwt.set_tuning(*before)


@pytest.mark.parametrize("choice", [(8, 6), (16, 8)])
@pytest.mark.parametrize("nb", [98_400, 131_100, 200_000, 400_000, 524_300, 600_000])
def test_no_level_is_left_to_the_host(nb, choice):
    cxbwt.set_tuning(*choice)
    rng = np.random.default_rng(nb)
    col = datagen.sample_reads(rng, datagen.random_genome(rng, nb // 20), nb // 100, 100, 0.005)
    _say(f"{choice}: {col.n_bases} bases")
    b, t = cxbwt.build_host(col.text, col.offsets)
    st = cxbwt.last_stats()
    assert st["host_levels"] == 0 and st["levels"] <= 3, (st["host_levels"], st["levels"])
    eb, et = oracle.bwt(col.text, col.offsets)
    assert np.array_equal(b, eb) and np.array_equal(t, et)


@pytest.mark.parametrize("count,size", [(4, 98_000), (4, 105_000), (3, 200_000), (2, 700_000)])
def test_batches_beyond_one_batch_of_scratch(count, size):
    # (of 105 and 200 kbases each: more segments than the scratch holds, known beforehand)
    cxbwt.set_tuning(*cxbwt.TUNING_CHOICES[0])
    rng = np.random.default_rng(size)
    cols = [datagen.sample_reads(rng, datagen.random_genome(rng, size // 20), size // 100, 100, 0.005)
            for _ in range(count)]
    _say(f"{count} collections of {size}")
    outs = cxbwt.build_batch_host(cols)
    for c, (b, t) in zip(cols, outs):
        eb, et = oracle.bwt(c.text, c.offsets)
        assert np.array_equal(b, eb) and np.array_equal(t, et)
