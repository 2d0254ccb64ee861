"""Small builds, whose levels are all enqueued before the host looks: at the
sizes where the number of levels changes, with inputs that need no further
level, that need more than were enqueued (the host completes them) and that
end in groups larger than a chunk.  Eager and replayed, against the oracle."""
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


def _lengths(rng, nb, lens):
    out = []
    while sum(out) < nb:
        out.append(int(rng.choice(lens)))
    out[-1] -= sum(out) - nb
    return np.array(out)


def _random(rng, nb):
    lens = _lengths(rng, nb, [60, 100, 101])
    return datagen.sample_reads(rng, datagen.random_genome(rng, max(200, nb // 8)), lens.size, lens, 0.01)


def _copies(rng, nb):
    one = "".join(datagen.ASCII[rng.integers(0, 4, size=90)].tobytes().decode())
    reads = [one] * (nb // 90) + [one[:nb % 90]]
    return datagen.from_reads([reads[i] for i in rng.permutation(len(reads))])


def _short(rng, nb):
    lens = _lengths(rng, nb, [1, 2, 3, 4, 5, 8])
    return datagen.random_collection(rng, lens.size, 1) if nb < 10 else datagen.Collection(
        datagen.ASCII[rng.integers(0, 2, size=nb)], np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64))


def _one_base(rng, nb):
    return datagen.from_reads(["A" * 120] * (nb // 120) + ["A" * (nb % 120)])


KINDS = {"random": _random, "copies": _copies, "short": _short, "one base": _one_base}


@pytest.mark.parametrize("choice", [(8, 6), (16, 8)])
@pytest.mark.parametrize("kind", list(KINDS))
def test_small_sizes(kind, choice):
    import torch
    cxbwt.set_tuning(*choice)
    chunk = 64 * choice[1]
    for nb in (1, chunk - 1, chunk, chunk + 1, 16 * chunk, 16 * chunk + 1, 256 * chunk, 256 * chunk + 7, 500_003):
        col = KINDS[kind](np.random.default_rng(nb), nb)
        assert col.n_bases == nb
        _say(f"{kind} {choice}: reads={col.n_reads} bases={nb}")
        eb, et = oracle.bwt(col.text, col.offsets)
        b, t = cxbwt.build_host(col.text, col.offsets)
        assert np.array_equal(b, eb) and np.array_equal(t, et), f"{kind} {nb}"
        packed, _ = cxbwt.pack(torch.from_numpy(col.text).cuda())
        off = torch.from_numpy(col.offsets.view(np.int64)).cuda()
        g = cxbwt.BuildGraph(packed, off, col.n_reads, nb, col.max_read_len)
        try:
            for _ in range(2):
                b, t = g.run()
                torch.cuda.synchronize()
                assert np.array_equal(b.cpu().numpy(), eb), f"{kind} {nb}: replay"
                assert np.array_equal(t.cpu().numpy().view(np.uint64), et), f"{kind} {nb}: replay"
        finally:
            g.close()
