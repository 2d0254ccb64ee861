"""What a user of this framework has it do, as cases that can be timed.

A pass is what a caller runs over reads that are already on the device: pack
the ASCII bases to 2-bit words and build the BWT and term_pos of the
collection(s), through the form of the entry point that fits the caller's
situation (caller's workspace, the library's fixed one, a captured graph, a
started job, a batch, key ranges).  The inputs are reads sampled from a random
genome on both strands with substitutions, the recipe of datagen, made on the
GPU from a seed.
"""
import math

import numpy as np
import torch

from paper_1401_7457_amd import cxbwt

#: 0 as tile/chunk: the calling thread's own choice (the library's default).
DEFAULTS = {"reads": 10_000, "len_min": 100, "len_max": 100, "coverage": 20.0, "error": 0.005, "repeats": False,
            "collections": 1, "budget": 0, "tile": 0, "chunk": 0}


def case(name, form, **kw):
    return {"name": name, "form": form, **DEFAULTS, **kw}


def listed():
    return [
        # a handful of reads (a local assembly, an interactive query): all latency
        case("few_reads", "noalloc", reads=63, len_min=100, len_max=250, error=0.01),
        # 1 Mbase, the smallest workload of the benchmark, in the library's fixed workspace
        case("one_megabase", "noalloc", reads=10_000, coverage=10.0, error=0.01),
        # the same size over and over (a serving loop of one shape): a captured graph replayed
        case("one_megabase_graph", "graph", reads=10_000, coverage=10.0, error=0.01),
        # one job of the server: reads of 100 to 250 bases, started and waited for
        case("served_job", "job", reads=50_021, len_min=100, len_max=250, coverage=8.0, error=0.01),
        # amplicon sequencing: a short target at very high depth, where most suffixes tie through whole reads
        case("deep_amplicon", "build", reads=200_003, len_min=100, len_max=100, coverage=2000.0, error=0.002),
        # many libraries of uneven size in one pass, the batched workload at a tenth of its collections
        case("batch", "batch", reads=1_500_000, len_min=75, len_max=150, coverage=12.0, collections=24),
        # a library built in key ranges because the workspace of a whole build does not fit the caller's budget
        case("key_ranges", "ranges", reads=2_000_000, coverage=20.0, budget=60_000_000),
        # longer reads at equal bases, the far end of the read-length sweep
        case("reads_400", "build", reads=500_000, len_min=400, len_max=400, coverage=20.0),
        # 4M reads of 100 bases at 20x (400 Mbases), the benchmark's second line with the choice its tuner makes
        case("plain_400m", "build", reads=4_000_000, coverage=20.0, tile=16, chunk=8),
        # the headline recipe, a repeat-heavy genome at 20x, at half its size: the largest whose state is held three times over
        case("repeats_2g", "build", reads=20_000_000, coverage=20.0, repeats=True, tile=16, chunk=8),
        # the packing alone: a loader that fills 2-bit buffers ahead of the builds
        case("pack_1g", "pack", reads=9_999_991),
    ]


def draw(rng):
    form = rng.choice(["noalloc", "build", "build", "build", "graph", "job", "batch", "ranges", "pack"])
    most = {"noalloc": 8e6, "graph": 2e8, "job": 3e8, "batch": 8e8, "ranges": 8e8, "pack": 1e9}.get(form, 1.5e9)
    least = {"batch": 2e6, "ranges": 2e6, "pack": 1e5}.get(form, 8e3)
    bases = math.exp(rng.uniform(math.log(least), math.log(most)))
    lo, hi = rng.choice([(100, 100), (100, 100), (75, 150), (100, 250), (150, 150), (35, 101), (200, 200), (400, 400)])
    reads = max(3, int(bases / ((lo + hi) / 2))) | 1
    deepest = 60.0 if bases > 1e8 else 2000.0
    tile, chunk = rng.choice([(0, 0), (0, 0), (8, 6), (16, 6), (16, 8)])
    if form not in ("build", "job", "batch"):
        tile = chunk = 0
    c = {"form": form, **DEFAULTS, "reads": reads, "len_min": lo, "len_max": hi,
         "coverage": round(math.exp(rng.uniform(math.log(5.0), math.log(deepest))), 2),
         "error": rng.choice([0.002, 0.005, 0.01]), "repeats": bases > 2e7 and rng.random() < 0.4,
         "tile": tile, "chunk": chunk}
    if form == "batch":
        c["collections"] = min(reads, int(math.exp(rng.uniform(math.log(2), math.log(256)))))
    if form == "ranges":
        c["budget"] = max(1000, int(reads * (lo + hi) / 2 / rng.choice([2.5, 4, 7])))
    return c


# --- inputs ------------------------------------------------------------------

def _collection_reads(c):
    """Reads per collection: log-uniform sizes over a factor of 100, summing to the case's reads."""
    k = c["collections"]
    if k == 1:
        return [c["reads"]]
    w = np.exp(np.random.default_rng(c["reads"] + k).uniform(0.0, math.log(100.0), size=k))
    r = np.maximum(1, np.floor(w / w.sum() * c["reads"]).astype(np.int64))
    r[int(np.argmax(r))] += c["reads"] - int(r.sum())
    return [int(x) for x in r]


def _mutated(codes, rate, gen):
    hit = torch.rand(codes.numel(), generator=gen, device="cuda") < rate
    step = torch.randint(1, 4, (codes.numel(),), generator=gen, device="cuda", dtype=torch.uint8)
    return torch.where(hit, (codes + step) & 3, codes)


def _genome(length, repeats, gen, host):
    """2-bit codes; with repeats, a tenth of it in families of 50 copies of 1 to 5 kb, each copy 1% diverged."""
    g = torch.randint(0, 4, (length,), generator=gen, device="cuda", dtype=torch.uint8)
    if not repeats or length < 2_000_000:
        return g
    units = []
    while sum(units) * 50 < length // 10:
        units.append(int(host.integers(1000, 5001)))
    starts = np.concatenate([[0], np.cumsum(units)])
    family = torch.randint(0, 4, (int(starts[-1]),), generator=gen, device="cuda", dtype=torch.uint8)
    piece = host.permutation(np.repeat(np.arange(len(units)), 50))
    size = np.asarray(units)[piece]
    cuts = np.sort(host.integers(0, length - int(size.sum()) + 1, size=piece.size))
    at = cuts + np.concatenate([[0], np.cumsum(size)[:-1]])
    size_d = torch.from_numpy(size).cuda()
    first = torch.repeat_interleave(torch.from_numpy(np.cumsum(size) - size).cuda(), size_d)
    inside = torch.arange(first.numel(), device="cuda") - first
    src = torch.repeat_interleave(torch.from_numpy(starts[piece]).cuda(), size_d) + inside
    dst = torch.repeat_interleave(torch.from_numpy(at).cuda(), size_d) + inside
    g[dst] = _mutated(family[src], 0.01, gen)
    return g


def _sample(text, base, lens, genome, error, gen):
    """Reads of the given lengths from both strands of the genome, written as ASCII at text[base:]."""
    ascii_of = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")
    n = lens.numel()
    for r0 in range(0, n, 1 << 20):
        L = lens[r0:r0 + (1 << 20)]
        start = (torch.rand(L.numel(), generator=gen, device="cuda", dtype=torch.float64) *
                 (genome.numel() - L + 1)).long()
        rev = torch.rand(L.numel(), generator=gen, device="cuda") < 0.5
        end = torch.cumsum(L, 0)
        total = int(end[-1])
        off = torch.repeat_interleave(start - (end - L), L) + torch.arange(total, device="cuda")
        flip = torch.repeat_interleave(rev, L)
        mirror = torch.repeat_interleave(2 * start + L - 1, L) - off
        codes = genome[torch.where(flip, mirror, off)]
        codes = _mutated(torch.where(flip, 3 - codes, codes), error, gen)
        text[base:base + total] = ascii_of[codes.long()]
        base += total
    return base


def _reads(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    host = np.random.default_rng(seed)
    per = _collection_reads(c)
    # the lengths a case holds are its own, their order the seed's (so that every seed has the same number of
    # bases): collections hold reads of one length each, a single one mixes its lengths
    if c["collections"] > 1:
        each = np.random.default_rng(c["reads"]).integers(c["len_min"], c["len_max"] + 1, size=len(per))
        lens = np.repeat(each, per)
    else:
        lens = c["len_min"] + np.arange(c["reads"]) % (c["len_max"] - c["len_min"] + 1)
        if c["len_max"] > c["len_min"]:
            lens = host.permutation(lens)
    offsets = np.zeros(lens.size + 1, dtype=np.int64)
    np.cumsum(lens, out=offsets[1:])
    text = torch.empty(int(offsets[-1]), dtype=torch.uint8, device="cuda")
    lens_d = torch.from_numpy(lens.astype(np.int64)).cuda()
    base, r0 = 0, 0
    for n in per:
        bases = int(offsets[r0 + n] - offsets[r0])
        genome = _genome(max(2 * c["len_max"], int(bases / c["coverage"])), c["repeats"], gen, host)
        base = _sample(text, base, lens_d[r0:r0 + n], genome, c["error"], gen)
        r0 += n
    bounds = np.concatenate([[0], np.cumsum(per)]).astype(np.uint64)
    return text, torch.from_numpy(offsets).cuda(), int(lens.max()), bounds


def prepare(c, seed):
    text, offsets, maxlen, bounds = _reads(c, seed)
    n, nb = offsets.numel() - 1, text.numel()
    s = {"form": c["form"], "text": text, "offsets": offsets, "n": n, "nb": nb, "maxlen": maxlen, "bounds": bounds,
         "budget": c["budget"], "opts": (c["tile"], c["chunk"], cxbwt.SCHEDULE_MSD) if c["tile"] else None,
         "packed": torch.empty(cxbwt.packed_words(nb), dtype=torch.int64, device="cuda"),
         "status": torch.empty(1, dtype=torch.int32, device="cuda")}
    if c["form"] == "pack":
        return s
    s["out"] = (torch.empty(nb + n, dtype=torch.uint8, device="cuda"), torch.empty(n, dtype=torch.int64, device="cuda"))
    if c["form"] == "noalloc":
        return s
    if c["form"] == "ranges":
        size = cxbwt.range_workspace_bytes(n, nb, maxlen, c["budget"])
    elif c["collections"] > 1:
        size = cxbwt.batch_workspace_bytes(n, nb, maxlen, c["collections"])
    else:
        size = cxbwt.workspace_bytes(n, nb, maxlen)
    s["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    if c["form"] == "graph":
        cxbwt.pack(text, out=s["packed"], status=s["status"])
        s["graph"] = cxbwt.BuildGraph(s["packed"], offsets, n, nb, maxlen, workspace=s["workspace"], out=s["out"])
    return s


def run(s):
    cxbwt.pack(s["text"], out=s["packed"], status=s["status"])
    form = s["form"]
    if form == "pack":
        return {"packed": s["packed"], "status": s["status"]}
    size = (s["packed"], s["offsets"], s["n"], s["nb"], s["maxlen"])
    if form == "noalloc":
        bwt, term = cxbwt.build_noalloc(*size, out=s["out"])
    elif form == "build":
        bwt, term = cxbwt.build(*size, workspace=s["workspace"], out=s["out"], opts=s["opts"])
    elif form == "job":
        bwt, term = cxbwt.build_start(*size, workspace=s["workspace"], out=s["out"], opts=s["opts"]).wait()
    elif form == "batch":
        bwt, term = cxbwt.build_batch(*size, s["bounds"], workspace=s["workspace"], out=s["out"], opts=s["opts"])
    elif form == "ranges":
        bwt, term = cxbwt.build_ranges(*size, s["budget"], workspace=s["workspace"], out=s["out"])
    else:
        bwt, term = s["graph"].run()
    return {"bwt": bwt, "term_pos": term}


def work(c):
    """The reads' bytes in; for a pack its words out, else the BWT and term_pos out and the offsets in."""
    n = c["reads"]
    nb = n * (c["len_min"] + c["len_max"]) / 2
    if c["form"] == "pack":
        return {"bytes": nb + nb / 4, "flops": 0.0}
    return {"bytes": nb + 8 * (n + 1) + (nb + n) + 8 * n, "flops": 0.0}


def exact(c, seed):
    """Every output is whole numbers, held bit for bit: no value in 64 bits stands beside them."""
    return None
