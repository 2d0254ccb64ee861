"""Builds in key ranges against the oracle where their levels can go wrong:
level 1 straight from the text with tiles of few members and of more than one
round's, prefixes below the first word of a key, 64-bit positions; later levels
whose chunks and final groups share the lists (chunks of 512) or do not."""
import sys
from collections import Counter

import numpy as np
import pytest

from oracle import oracle
from paper_1401_7457_amd import cxbwt, datagen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    cxbwt.lib()
    before = cxbwt.get_tuning()
    yield
    cxbwt.set_tuning(*before)


def _deep(rng):
    # ties through whole reads, and groups of identical suffixes level after level
    col = datagen.sample_reads(rng, datagen.random_genome(rng, 1500), 12_000, rng.choice([33, 60, 100], size=12_000), 0.002)
    return col


def _few_keys(rng):
    # most suffixes in a few prefixes: prefixes of many digits, pieces of one class
    text = datagen.ASCII[np.where(rng.random(700_000) < 0.02, 3, 0)]
    return datagen.Collection(text, np.arange(0, 700_001, 70, dtype=np.uint64))


def _ragged(rng):
    return datagen.random_collection(rng, 9000, [0, 1, 2, 26, 27, 28, 53, 55, 150])


def _largest_class(col):
    """Most suffixes that share a whole first window (27 bases)."""
    text, counts = col.text.tobytes(), Counter()
    for a, b in zip(col.offsets[:-1].tolist(), col.offsets[1:].tolist()):
        counts.update(text[i:i + 27] for i in range(a, b - 26))
    return max(counts.values(), default=0)


@pytest.mark.parametrize("tuning", [(16, 8), (8, 6)])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("share", [0.93, 0.3, 0.05])
@pytest.mark.parametrize("shape", [_deep, _few_keys, _ragged])
def test_ranges_equal_the_oracle(shape, share, wide, tuning):
    col = shape(np.random.default_rng(3))
    cxbwt.set_tuning(*tuning)
    m = int(col.n_bases * share)
    print(f"[case] {shape.__name__} bases={col.n_bases} budget={m} wide={wide} tuning={tuning}", flush=True)
    sys.stdout.flush()
    if _largest_class(col) > m:  # suffixes that agree in a whole window are one range
        with pytest.raises(cxbwt.CxbwtError) as e:
            cxbwt.build_host(col.text, col.offsets, max_range_suffixes=m, wide=wide)
        assert e.value.status == cxbwt.ERANGE
        return
    b, t = cxbwt.build_host(col.text, col.offsets, max_range_suffixes=m, wide=wide)
    eb, et = oracle.bwt(col.text, col.offsets)
    assert np.array_equal(b, eb)
    assert np.array_equal(t, et)
