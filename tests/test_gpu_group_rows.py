"""Groups of identical suffixes far larger than a tile, in builds small enough
to list their levels: right, and written by many workgroups."""
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
    before = cxbwt.set_timing(True)
    yield
    cxbwt.set_timing(before)


@pytest.mark.parametrize("reads,length", [(4_000_000, 1), (250_000, 25)])
def test_rows_of_large_groups(reads, length):
    # single bases: four groups of a million; copies of one read: a group per suffix
    rng = np.random.default_rng(length)
    if length == 1:
        text = datagen.ASCII[rng.integers(0, 4, size=reads)]
    else:
        text = np.tile(datagen.ASCII[rng.integers(0, 4, size=length)], reads)
    offsets = np.arange(0, text.size + 1, length, dtype=np.uint64)
    _say(f"reads={reads} of {length}")
    ms = []
    for _ in range(3):
        b, t = cxbwt.build_host(text, offsets)
        ms.append(cxbwt.last_stats()["ms"]["final_emit"])
    rc = oracle.check_bwt(b, t, text, offsets)
    assert rc == 0, f"invariant {rc} fails"
    # one workgroup writes a million rows in about 4 ms (a quarter of a million
    # in about 1), all of them the whole in a tenth of that
    assert min(ms) < (1.5 if length == 1 else 0.5), ms
