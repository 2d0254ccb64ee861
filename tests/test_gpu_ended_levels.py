"""The levels that split off the suffixes ending at a digit, on reads full of
the base whose digits are all zero: the oracle's result, and no more levels
than the digits need once such a split has found few suffixes ending."""
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


def _runs_inside(rng, n, length, run, every):
    col = datagen.sample_reads(rng, datagen.random_genome(rng, 40_000), n, length, 0.005)
    text = col.text.reshape(n, length)
    text[::every, 4:4 + run] = ord("A")
    return col


def _few_other_bases(rng, n, length):
    codes = np.where(rng.random(n * length) < 0.01, rng.integers(1, 4, size=n * length), 0)
    return datagen.Collection(datagen.ASCII[codes], np.arange(0, n * length + 1, length, dtype=np.uint64))


CASES = {"runs": lambda rng: _runs_inside(rng, 10_000, 100, 90, 10),
         "nearly one base": lambda rng: _few_other_bases(rng, 8_000, 100),
         "ends at every digit": lambda rng: datagen.from_reads(
             ["ACGT"[i % 3 + 1] * (i % 2) + "A" * int(k) for i, k in enumerate(rng.integers(1, 60, size=30_000))])}


@pytest.mark.parametrize("case", list(CASES))
def test_levels_of_zero_digits(case):
    col = CASES[case](np.random.default_rng(17))
    _say(f"{case}: reads={col.n_reads} bases={col.n_bases}")
    b, t = cxbwt.build_host(col.text, col.offsets)
    st = cxbwt.last_stats()
    eb, et = oracle.bwt(col.text, col.offsets)
    assert np.array_equal(b, eb) and np.array_equal(t, et)
    # eight digits a window of 27 bases; and a split before it for every digit
    # that suffixes end at, which a level more each when an eighth and more do
    # (a chunk is 384 of at most 1.1 million), once when they do not
    windows = col.max_read_len // 27 + 1
    spare = 1 if case == "runs" else 7 * windows
    assert st["levels"] <= 8 * windows + spare, st["levels"]
