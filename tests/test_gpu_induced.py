"""Builds large enough to sort only the samples of their suffixes and derive
the order of the others, at the shapes where that can go wrong: ragged and
empty reads, runs around the regions and beyond them, collections without
samples, small ones among large, tie groups above a chunk.  Checked by the
properties that fix a BWT (counts, terminator rows, the LF walk of every read)."""
import sys

import numpy as np
import pytest

from oracle import oracle
from paper_1401_7457_amd import cxbwt, datagen

pytestmark = pytest.mark.gpu

SIZE = 34_000_000  # bases: above the size from which the samples alone are sorted


def _say(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    cxbwt.lib()


def _with_runs(col, rng, lengths, every):
    """Every `every`-th read gets a run of one base written over it."""
    for i in range(0, col.n_reads, every):
        a, b = int(col.offsets[i]), int(col.offsets[i + 1])
        k = int(rng.choice(lengths))
        if b - a > k + 2:
            at = a + int(rng.integers(0, b - a - k))
            col.text[at:at + k] = datagen.ASCII[int(rng.integers(4))]
    return col


def _ragged(rng):
    lens = rng.choice([0, 1, 2, 15, 16, 17, 22, 23, 47, 60, 100, 101, 150, 333], size=SIZE // 60)
    return datagen.sample_reads(rng, datagen.random_genome(rng, 2_000_000), lens.size, lens, 0.01)


def _runs(rng):
    col = datagen.sample_reads(rng, datagen.random_genome(rng, 2_000_000), SIZE // 100, 100, 0.005)
    return _with_runs(col, rng, [13, 14, 15, 16, 17, 18, 19], 5000)


def _two_letters(rng):
    n = SIZE // 80
    text = datagen.ASCII[np.where(rng.random(n * 80) < 0.3, 3, 2)]
    return _with_runs(datagen.Collection(text, np.arange(0, n * 80 + 1, 80, dtype=np.uint64)), rng, [2], 1)


def _deep(rng):
    return datagen.sample_reads(rng, datagen.random_genome(rng, 12_000), SIZE // 100, 100, 0.001)


def _long_runs(rng):
    # runs the steps would follow too far: sorted whole
    col = datagen.sample_reads(rng, datagen.random_genome(rng, 2_000_000), SIZE // 400, 400, 0.005)
    return _with_runs(col, rng, [300, 390], 50)


CASES = {"ragged": _ragged, "runs": _runs, "two letters": _two_letters, "deep": _deep, "long runs": _long_runs}


@pytest.mark.parametrize("case", list(CASES))
def test_induced_build(case):
    col = CASES[case](np.random.default_rng(sum(map(ord, case))))
    _say(f"{case}: reads={col.n_reads} bases={col.n_bases}")
    b, t = cxbwt.build_host(col.text, col.offsets)
    rc = oracle.check_bwt(b, t, col.text, col.offsets)
    assert rc == 0, f"{case}: invariant {rc} fails"


def test_induced_batch_of_uneven_collections():
    rng = np.random.default_rng(5)
    cols = [_with_runs(datagen.sample_reads(rng, datagen.random_genome(rng, 50_000 + 1000 * k), n, L, 0.01), rng,
                       [14, 15, 16], 900)
            for k, (n, L) in enumerate([(3, 50), (200_000, 75), (1, 40), (90_000, 100), (7, 100), (5000, 150), (60_000, 101)])]
    cols.insert(2, datagen.from_reads(["ACGTACGT" * 12] * 500))
    cols.insert(4, datagen.from_reads(["A" * 14, "C" * 12, "TTTT", ""] * 300))  # no samples at all
    cols.append(datagen.from_reads(["T" * 9 + "G" * 9 + "C" * 9] * 900))          # none either
    _say(f"batch: {[c.n_bases for c in cols]}")
    assert sum(c.n_bases for c in cols) >= SIZE * 0.9
    for i, (c, (b, t)) in enumerate(zip(cols, cxbwt.build_batch_host(cols))):
        assert oracle.check_bwt(b, t, c.text, c.offsets) == 0, f"collection {i}"


@pytest.mark.parametrize("tuning", [(8, 3), (6, 6)])
def test_sorted_whole_under_a_chosen_tuning(tuning):
    # the sort that follows a declined induction has its own tiles
    col = _long_runs(np.random.default_rng(5))
    before = cxbwt.get_tuning()
    try:
        cxbwt.set_tuning(*tuning)
        _say(f"long runs, tuning {tuning}: reads={col.n_reads} bases={col.n_bases}")
        b, t = cxbwt.build_host(col.text, col.offsets)
        st = cxbwt.last_stats()
    finally:
        cxbwt.set_tuning(*before)
    assert st["chunk_suffixes"] > col.n_bases // 2  # sorted whole
    rc = oracle.check_bwt(b, t, col.text, col.offsets)
    assert rc == 0, f"invariant {rc} fails"


@pytest.mark.parametrize("lens", [[160], [161], [22, 47, 64, 65, 66, 108, 161, 151], [300]])
def test_windows_of_long_reads(lens):
    # ties that last to the reads' ends, which fall on and beside the ends of
    # the windows (22, then 25 and 18 in turn) of the reads that take two at once
    rng = np.random.default_rng(lens[0] + len(lens))
    n = int(SIZE // np.mean(lens))
    col = datagen.sample_reads(rng, datagen.random_genome(rng, 40_000), n, rng.choice(lens, size=n), 0.001)
    _say(f"lengths {lens}: reads={col.n_reads} bases={col.n_bases}")
    b, t = cxbwt.build_host(col.text, col.offsets)
    rc = oracle.check_bwt(b, t, col.text, col.offsets)
    assert rc == 0, f"invariant {rc} fails"


def test_batch_sorted_whole_among_small_collections():
    # long runs in one collection: the sort takes all above one chunk, and the
    # small ones are finished once
    rng = np.random.default_rng(8)
    cols = [datagen.random_collection(rng, 3, [40]), _long_runs(rng), datagen.random_collection(rng, 4, [50]),
            datagen.sample_reads(rng, datagen.random_genome(rng, 20_000), 2000, 75, 0.01)]
    _say(f"batch: {[c.n_bases for c in cols]}")
    outs = cxbwt.build_batch_host(cols)
    st = cxbwt.last_stats()
    assert st["chunk_suffixes"] > cols[1].n_bases // 2  # sorted whole
    for i, (c, (b, t)) in enumerate(zip(cols, outs)):
        assert oracle.check_bwt(b, t, c.text, c.offsets) == 0, f"collection {i}"
    # the chunks are those of the collections above one chunk, and one each of the small
    cxbwt.build_batch_host([cols[1], cols[3]])
    assert st["chunks"] == cxbwt.last_stats()["chunks"] + 2
