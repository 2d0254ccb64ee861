"""A graph of the default number of levels is complete in stream order: after
launch and a stream wait the outputs are the oracle's, for contents that need
far more levels than those at capture, before finish is called."""
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


def _put(text, offsets):
    import torch
    packed, status = cxbwt.pack(torch.from_numpy(np.ascontiguousarray(text)).cuda())
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    return packed, torch.from_numpy(offsets.view(np.int64)).cuda()


def _deeper(rng, n, length):
    """Contents of the same shape: ties through whole reads, and digits that are
    zero but for a few reads, so that every digit of every window is a level."""
    rare = np.where(rng.random(n * length) < 0.01, rng.integers(1, 4, size=n * length), 0)
    genome = datagen.random_genome(rng, length + 10)  # few groups: one batch a level
    yield "nearly one base", datagen.ASCII[rare]
    yield "one base", np.full(n * length, ord("A"), dtype=np.uint8)
    yield "a short genome", datagen.sample_reads(rng, genome, n, length, 0.002).text


@pytest.mark.parametrize("choice,n,collections", [((8, 6), 6000, 1), ((16, 8), 6000, 1), ((8, 3), 6000, 1),
                                                  ((8, 6), 1500, 3)])
def test_outputs_after_launch_alone(choice, n, collections):
    import torch
    rng = np.random.default_rng(23)
    length = 100
    cxbwt.set_tuning(*choice)
    shallow = datagen.sample_reads(rng, datagen.random_genome(rng, 10 * n), n, length, 0.01)
    packed, offs = _put(shallow.text, shallow.offsets)
    bounds = np.linspace(0, n, collections + 1).astype(np.uint64)
    g = cxbwt.BuildGraph(packed, offs, n, n * length, length, coll_reads=bounds)
    try:
        for label, text in [("as captured", shallow.text), *_deeper(rng, n, length), ("as captured", shallow.text)]:
            if label == "a short genome" and (choice[1] == 3 or collections > 1):
                continue  # more segments above a chunk than the scratch holds in one batch: the host's to finish
            g.packed.copy_(_put(text, shallow.offsets)[0])
            _say(f"{choice}, {collections} collections, {label}: launch")
            g.bwt.fill_(0)
            g.term.fill_(0)
            g.launch()
            torch.cuda.synchronize()
            b, t = g.bwt.cpu().numpy().copy(), g.term.cpu().numpy().copy()
            g.finish()
            st = cxbwt.last_stats()
            assert st["host_levels"] == 0, f"{label}: {st['host_levels']} levels were left to the host"
            for c in range(collections):
                r0, r1 = int(bounds[c]), int(bounds[c + 1])
                eb, et = oracle.bwt(text[r0 * length:r1 * length], shallow.offsets[r0:r1 + 1] - shallow.offsets[r0])
                got = b[r0 * (length + 1):r1 * (length + 1)]
                assert np.array_equal(got, eb), f"{label}: collection {c}"
                assert np.array_equal(t[r0:r1].view(np.uint64), et), f"{label}: collection {c}"
            eager = cxbwt.build_batch(g.packed, offs, n, n * length, length, bounds)  # eager work in between
            torch.cuda.synchronize()
            assert np.array_equal(eager[0].cpu().numpy(), b)
    finally:
        g.close()
