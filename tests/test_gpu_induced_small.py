"""The build by induced order, row by row against the oracle, on many random
collections: run in a build of the library that takes it from 60 000 bases on.
Every case says that it was taken (half of the suffixes at most are sorted) or
that it was declined."""
import sys

import numpy as np
import pytest

from oracle import oracle
from paper_1401_7457_amd import build, cxbwt, datagen

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(autouse=True)
def small_library(monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    monkeypatch.setattr(cxbwt, "LIB_PATH", build.SMALL_OUT)
    monkeypatch.setattr(cxbwt, "_lib", None)
    cxbwt.lib()


def _collection(text, lens):
    offsets = np.zeros(len(lens) + 1, dtype=np.uint64)
    np.cumsum(np.asarray(lens, dtype=np.uint64), out=offsets[1:])
    return datagen.Collection(np.ascontiguousarray(text[:int(offsets[-1])]), offsets)


def _with_runs(col, rng, lengths, count):
    """Runs of one base written over `count` reads that hold them."""
    size = np.diff(col.offsets.astype(np.int64))
    for i in rng.choice(np.flatnonzero(size > max(lengths) + 2), size=count):
        a, k = int(col.offsets[i]), int(rng.choice(lengths))
        at = a + int(rng.integers(0, size[i] - k))
        col.text[at:at + k] = datagen.ASCII[int(rng.integers(4))]
    return col


def _ragged(rng, nb):
    lens = rng.choice([0, 1, 2, 7, 15, 16, 17, 21, 22, 23, 44, 47, 48, 60, 65, 100, 101, 150], size=nb // 40)
    return datagen.sample_reads(rng, datagen.random_genome(rng, nb // 10), lens.size, lens, 0.01)


def _short(rng, nb):
    # one read reaches the length from which the samples are sorted
    lens = np.concatenate([rng.integers(0, 30, size=nb // 14), [40]])
    return _collection(datagen.ASCII[rng.integers(0, 4, size=int(lens.sum()))], lens)


def _two_letters(letters):
    def make(rng, nb):
        lens = rng.integers(20, 80, size=nb // 50)
        # runs of at most 12 on their own, every letter in many of them
        text = datagen.ASCII[rng.choice(letters, size=int(lens.sum()))]
        text[11::12] = datagen.ASCII[letters[0]]
        text[5::12] = datagen.ASCII[letters[1]]
        return _collection(text, lens)
    return make


def _runs(rng, nb):
    # around the run regions, past them, and past the 32 positions of a record
    # pair; too few steps beyond the regions to be declined
    col = datagen.sample_reads(rng, datagen.random_genome(rng, nb // 10), nb // 100, 100, 0.005)
    return _with_runs(col, rng, [12, 13, 14, 15, 16, 17], nb // 4000)


def _long_run(base):
    def make(rng, nb):
        col = datagen.sample_reads(rng, datagen.random_genome(rng, nb // 10), nb // 100, 100, 0.005)
        for i in range(3, col.n_reads, 400):  # at every offset of a record
            a = int(col.offsets[i]) + i % 16
            col.text[a:a + 25] = ord(base)
        return col
    return make


def _deep(rng, nb):
    # tie groups above a chunk, whole reads among them
    return datagen.sample_reads(rng, datagen.random_genome(rng, 400), nb // 80, rng.choice([60, 80, 100], size=nb // 80),
                                0.002)


def _long_reads(rng, nb):
    lens = rng.choice([161, 300, 47, 90], size=nb // 150)
    return datagen.sample_reads(rng, datagen.random_genome(rng, nb // 40), lens.size, lens, 0.002)


CASES = {"ragged": _ragged, "short": _short, "A and C": _two_letters([0, 1]), "G and T": _two_letters([2, 3]),
         "T and A": _two_letters([3, 0]), "runs": _runs, "long A": _long_run("A"), "long C": _long_run("C"),
         "long T": _long_run("T"), "deep": _deep, "long reads": _long_reads}


def _check(col, b, t, label):
    eb, et = oracle.bwt(col.text, col.offsets)
    if not np.array_equal(b, eb):
        bad = np.flatnonzero(b != eb)
        raise AssertionError(f"{label}: {bad.size} BWT rows differ, first {bad[:10].tolist()}")
    assert np.array_equal(t, et), f"{label}: term_pos differs"


@pytest.mark.parametrize("nb", [100_000, 262_144, 700_001])
@pytest.mark.parametrize("case", list(CASES))
def test_rows_against_the_oracle(case, nb):
    for seed in range(3):
        col = CASES[case](np.random.default_rng(1000 * seed + nb), nb)
        _say(f"{case} {nb} seed {seed}: reads={col.n_reads} bases={col.n_bases}")
        b, t = cxbwt.build_host(col.text, col.offsets)
        st = cxbwt.last_stats()
        assert st["chunk_suffixes"] <= col.n_bases // 2, "declined"
        _check(col, b, t, f"{case} {nb} {seed}")


@pytest.mark.parametrize("seed", range(3))
def test_batches_against_the_oracle(seed):
    rng = np.random.default_rng(seed)
    kinds = list(CASES.values())
    cols = [kinds[int(k)](rng, int(nb)) for k, nb in zip(rng.permutation(len(kinds)),
                                                          np.exp(rng.uniform(np.log(8_000), np.log(200_000), 11)))]
    cols.insert(1, datagen.from_reads(["ACGT", "", "TT"]))
    cols.insert(4, datagen.from_reads(["A" * 14, "C" * 12, "TTTT", ""] * 300))  # no samples
    cols.append(datagen.from_reads(["T" * 9 + "G" * 9 + "C" * 9] * 900))          # none either
    _say(f"batch {seed}: {[c.n_bases for c in cols]}")
    outs = cxbwt.build_batch_host(cols)
    assert cxbwt.last_stats()["chunk_suffixes"] <= sum(c.n_bases for c in cols) // 2, "declined"
    for i, (c, (b, t)) in enumerate(zip(cols, outs)):
        _check(c, b, t, f"collection {i}")


def test_the_bound_on_read_lengths_chooses_nothing():
    # the bound may be any number above the lengths: the same kernels, the same loads
    col = _deep(np.random.default_rng(6), 200_000)
    loads = []
    for bound in (100, 161, 400, 65_535):
        _say(f"bound {bound}")
        b, t = cxbwt.build_host(col.text, col.offsets, max_read_len=bound)
        loads.append(cxbwt.last_stats()["window_fetches"])
        _check(col, b, t, f"bound {bound}")
    assert len(set(loads)) == 1, loads


def test_declined_builds_are_sorted():
    col = _with_runs(datagen.sample_reads(np.random.default_rng(3), datagen.random_genome(np.random.default_rng(4), 20_000),
                                          2000, 100, 0.005), np.random.default_rng(5), [70, 90], 100)
    _say(f"long runs: reads={col.n_reads} bases={col.n_bases}")
    b, t = cxbwt.build_host(col.text, col.offsets)
    assert cxbwt.last_stats()["chunk_suffixes"] > col.n_bases // 2
    _check(col, b, t, "long runs")


@pytest.mark.parametrize("large", ["none", "induced", "declined"])
def test_many_small_collections_are_sorted(large):
    """More than 400 collections that one level sorts, alone, beside large ones
    and beside one whose induction is declined: they are sorted whole."""
    rng = np.random.default_rng(11)
    cols = [datagen.sample_reads(rng, datagen.random_genome(rng, 300), n, 50, 0.01)
            for n in rng.choice([2, 5, 20, 60, 120], size=800)]
    small = sum(c.n_bases for c in cols)
    if large != "none":
        for k, at in enumerate((0, 300, 802)):
            c = datagen.sample_reads(rng, datagen.random_genome(rng, 20_000), 1500 + 100 * k, 100, 0.005)
            cols.insert(at, _with_runs(c, rng, [60, 90], 40) if large == "declined" and k == 1 else c)
    total = sum(c.n_bases for c in cols)
    _say(f"{large}: {len(cols)} collections, {total} bases")
    outs = cxbwt.build_batch_host(cols)
    st = cxbwt.last_stats()
    final = {"none": total, "induced": small + (total - small) // 2, "declined": total}[large]
    assert st["chunk_suffixes"] <= final and st["chunk_suffixes"] >= (small if large == "induced" else 0.9 * total)
    for i, (c, (b, t)) in enumerate(zip(cols, outs)):
        _check(c, b, t, f"collection {i}")


def test_two_induced_builds_in_flight():
    """Started on two streams, each waiting for its own levels: four rounds, so
    that the host blocks and events go round."""
    import torch
    cols = [_deep(np.random.default_rng(1), 300_000), _ragged(np.random.default_rng(2), 500_000)]
    streams = [torch.cuda.Stream() for _ in cols]
    sides = []
    for c, s in zip(cols, streams):
        with torch.cuda.stream(s):
            packed, _ = cxbwt.pack(torch.from_numpy(c.text).cuda())
            offs = torch.from_numpy(c.offsets.view(np.int64)).cuda()
        sides.append((c, s, packed, offs))
    torch.cuda.synchronize()
    for k in range(4):
        jobs = [(c, cxbwt.build_start(p, o, c.n_reads, c.n_bases, c.max_read_len, stream=s)) for c, s, p, o in sides]
        for c, j in jobs:
            b, t = j.wait()
            torch.cuda.synchronize()
            assert j.stats["chunk_suffixes"] <= c.n_bases // 2, "declined"
            _check(c, b.cpu().numpy(), t.cpu().numpy().view(np.uint64), f"round {k}")
