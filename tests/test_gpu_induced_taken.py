"""Which builds of the library sort samples only: from 16.5 Mbases on, with a
read above 32 bases, and of a batch the large collections; seen in the
statistics (a build that sorts every suffix gives the same rows)."""
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


def _reads(n, length):
    rng = np.random.default_rng(n)
    return datagen.sample_reads(rng, datagen.random_genome(rng, n * length // 20), n, length, 0.005)


@pytest.mark.parametrize("n,length,taken", [(164_900, 100, False), (165_100, 100, True), (520_000, 32, False),
                                            (502_000, 33, True)])
def test_sizes(n, length, taken):
    col = _reads(n, length)
    _say(f"reads={n} of {length}")
    b, t = cxbwt.build_host(col.text, col.offsets)
    st = cxbwt.last_stats()
    assert (st["chunk_suffixes"] <= col.n_bases // 2) == taken, st["chunk_suffixes"]
    assert oracle.check_bwt(b, t, col.text, col.offsets) == 0


def test_batch():
    large, small = _reads(170_000, 100), [_reads(30, 100) for _ in range(450)]
    _say("one collection of 17 Mbases among 450 of 3 kbases")
    outs = cxbwt.build_batch_host([large, *small])
    st = cxbwt.last_stats()
    rest = sum(c.n_bases for c in small)
    assert rest <= st["chunk_suffixes"] <= rest + large.n_bases // 2
    for c, (b, t) in zip([large, small[0], small[-1]], [outs[0], outs[1], outs[-1]]):
        assert oracle.check_bwt(b, t, c.text, c.offsets) == 0
