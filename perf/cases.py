"""The scans that a user of the library runs, as cases to be timed.

A case names a call, a pattern set and the texts it scans.  Pattern sets and
texts follow the workloads c1 .. c5 of ``synth`` (random signatures over all
bytes or mostly printable bytes, DNA reads, batches of packets and files,
served requests) and two sets that the general kernels serve: dictionary words
over lower-case text, whose matches are dense, and short DNA motifs.

Fields of a case
  call      scan | scan_sync | scan_noalloc | batch | graph | serve
  dist      uniform | mix | acgt | words: bytes of the patterns and the text
  k, lo, hi patterns and the range of their lengths
  n         bytes of the text (scan, scan_sync, scan_noalloc)
  gap       mean distance of planted copies of patterns in bytes
  shift     bytes the text's address lies past a 256-byte boundary
  counts    per-position counts are asked for as well
  small, median, large, large_lo, large_hi   (batch, graph, serve) number of
            small texts and their median length, number of large texts and the
            range of their lengths

Every output is whole numbers (match records, counts), so there is no value
in 64 bits to compare with: records stay equal, byte by byte.
"""

import math
import types

import numpy as np
import torch

import paper_1702_03657_amd as pf

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
RECORD = 16  # bytes of a match record

# lower-case letters by their frequency in English prose (per mille)
LETTERS = np.array([82, 15, 28, 43, 127, 22, 20, 61, 70, 2, 8, 40, 24, 67, 75, 19, 1, 60, 63, 91, 28, 10, 24, 2, 20, 1],
                   dtype=np.float64)
VOCABULARY = 20_000  # words of the lower-case text


def _one(name, call, dist, k, lo, hi, n, gap, shift=0, counts=False):
    return dict(name=name, call=call, dist=dist, k=k, lo=lo, hi=hi, n=n, gap=gap, shift=shift, counts=counts)


def _many(name, call, dist, k, lo, hi, gap, small, median, large=0, large_lo=0, large_hi=0):
    return dict(name=name, call=call, dist=dist, k=k, lo=lo, hi=hi, gap=gap, small=small, median=median,
                large=large, large_lo=large_lo, large_hi=large_hi)


def listed():
    return [
        # one packet against a signature set, the count wanted on the host:
        # launches and the synchronisation are all there is
        _one("packet_1460", "scan_sync", "mix", 1000, 8, 64, 1460, 512),
        # a small file against a few short signatures (c1)
        _one("file_1m", "scan", "uniform", 100, 4, 16, 1 * MiB, 1024),
        # a log of odd size at an odd address, with per-position counts
        _one("log_5m_counts", "scan", "mix", 10_000, 8, 64, 5_000_011, 4096, shift=3, counts=True),
        # a file scanned by code that cannot allocate
        _one("blob_24m_noalloc", "scan_noalloc", "uniform", 20_000, 8, 64, 24_000_007, 2048),
        # keywords of a dictionary in prose: about one match per 100 bytes
        _one("words_16m", "scan", "words", 2000, 4, 12, 16 * MiB + 77, 4096),
        # a large file against a signature set (c2)
        _one("signatures_256m", "scan", "mix", 10_000, 8, 64, 256 * MiB, 4096),
        # a genome against sequenced reads (c3)
        _one("dna_1g", "scan", "acgt", 100_000, 20, 32, 1 * GiB, 100_000),
        # short motifs in a chromosome: too short for the 16-symbol filter
        _one("motifs_32m", "scan", "acgt", 500, 9, 14, 32 * MiB + 5, 8192),
        # a few hundred documents gathered for one scan
        _many("documents_batch", "batch", "mix", 5000, 6, 48, 4096, 600, 1024, 12, 64 * KiB, 512 * KiB),
        # a second of packets, scanned by replaying a graph (c4's small texts)
        _many("packets_graph", "graph", "uniform", 20_000, 8, 64, 2048, 65_536, 512),
        # packets and files mixed (c4), the largest work
        _many("mixed_graph", "graph", "uniform", 20_000, 8, 64, 2048, 65_536, 512, 64, 1 * MiB, 64 * MiB),
        # requests in host memory through the server (c5's sizes up to 4 MiB)
        _many("serve_24", "serve", "uniform", 10_000, 8, 64, 2048, 12, 4096, 12, 64 * KiB, 4 * MiB),
    ]


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["packet", "file", "file", "blob", "words", "large", "dna", "motifs", "documents", "packets",
                       "mixed", "serve"])
    shift = rng.choice([0, 0, 1, 3, 8, 13])
    dist = rng.choice(["mix", "uniform"])
    if kind == "packet":
        c = _one("", "scan_sync", dist, log(100, 10_000), 8, 64, log(64, 64 * KiB), 512, shift)
    elif kind == "file":
        c = _one("", "scan", dist, log(50, 10_000), rng.choice([4, 6, 8]), rng.choice([16, 32, 64]),
                 log(64 * KiB, 8 * MiB), rng.choice([1024, 4096]), shift, rng.random() < 0.3)
    elif kind == "blob":
        c = _one("", rng.choice(["scan_noalloc", "scan"]), dist, log(1000, 20_000), 8, 64, log(4 * MiB, 30 * MiB), 2048,
                 shift)
    elif kind == "words":
        c = _one("", "scan", "words", log(200, 2000), rng.choice([4, 5]), rng.choice([10, 12]), log(256 * KiB, 16 * MiB),
                 4096, shift)
    elif kind == "large":
        c = _one("", "scan", dist, log(1000, 20_000), 8, 64, log(16 * MiB, 256 * MiB), 4096, shift)
    elif kind == "dna":
        c = _one("", "scan", "acgt", log(1000, 100_000), 20, 32, log(16 * MiB, 1 * GiB), 100_000, shift)
    elif kind == "motifs":
        c = _one("", "scan", "acgt", log(50, 500), rng.choice([9, 10]), rng.choice([12, 14]), log(1 * MiB, 32 * MiB),
                 8192, shift)
    elif kind == "documents":
        c = _many("", rng.choice(["batch", "graph"]), dist, log(500, 10_000), 6, 48, 4096, log(20, 1000), log(256, 1400),
                  rng.randint(0, 12), 64 * KiB, 512 * KiB)
    elif kind == "packets":
        c = _many("", rng.choice(["batch", "graph"]), "uniform", log(2000, 20_000), 8, 64, 2048, log(2000, 65_536),
                  rng.choice([128, 512, 900]))
    elif kind == "mixed":
        c = _many("", "graph", dist, log(2000, 20_000), 8, 64, 2048, log(1000, 65_536), 512, rng.randint(4, 32), 1 * MiB,
                  log(4 * MiB, 48 * MiB))
    else:
        c = _many("", "serve", "uniform", log(1000, 10_000), 8, 64, 2048, rng.randint(2, 14), 4096, rng.randint(2, 14),
                  64 * KiB, log(256 * KiB, 4 * MiB))
    del c["name"]
    return c


# ------------------------------------------------------------------- inputs


def _lengths(case):
    """Lengths of the texts of a batch, the same for every seed: a batch's
    size belongs to the case, its bytes to the seed."""
    rng = np.random.default_rng([case["small"], case["median"], case["large"], case["large_lo"], case["large_hi"]])
    top = 1500 if case["call"] != "serve" else 64 * KiB
    small = np.clip(np.rint(rng.lognormal(math.log(case["median"]), 0.75, case["small"])), 64, top).astype(np.int64)
    large = rng.integers(case["large_lo"], case["large_hi"] + 1, case["large"])
    lens = np.concatenate([small, large])
    return lens[rng.permutation(len(lens))]


def _total(case):
    return case["n"] if "n" in case else int(_lengths(case).sum())


def _expected(case):
    """Matches to expect, for the size of the output."""
    n = _total(case)
    m = n / case["gap"]
    if case["dist"] == "words":
        m += n / 100
    elif case["dist"] == "acgt":
        m += n * case["k"] * 4.0 ** -case["lo"] / 3 / (case["hi"] - case["lo"] + 1) * 4
    return m


def _vocabulary(rng):
    lens = rng.integers(2, 13, VOCABULARY)
    letters = (97 + rng.choice(26, int(lens.sum()), p=LETTERS / LETTERS.sum())).astype(np.uint8)
    return letters, lens


def _patterns(case, rng, vocabulary):
    lo, hi, k = case["lo"], case["hi"], case["k"]
    if case["dist"] == "words":
        letters, lens = vocabulary
        start = np.cumsum(lens) - lens
        # not the commonest words: they are not what one searches for
        fit = np.nonzero((lens >= lo) & (lens <= hi))[0]
        ids = rng.choice(fit[fit >= 100], k, replace=False)
        data = np.concatenate([letters[start[i]:start[i] + lens[i]] for i in ids])
        plen = lens[ids]
    else:
        plen = rng.integers(lo, hi + 1, k)
        m = int(plen.sum())
        if case["dist"] == "acgt":
            data = np.frombuffer(b"ACGT", dtype=np.uint8)[rng.integers(0, 4, m)]
        elif case["dist"] == "mix":
            data = np.where(rng.random(m) < 0.7, rng.integers(0x20, 0x7F, m), rng.integers(0, 256, m)).astype(np.uint8)
        else:
            data = rng.integers(0, 256, m, dtype=np.uint8)
    offsets = np.zeros(k + 1, dtype=np.uint64)
    offsets[1:] = np.cumsum(plen)
    return types.SimpleNamespace(data=data, offsets=offsets)


def _text(case, n, gen, vocabulary, out):
    """Fill the device tensor `out` (n bytes) with text."""
    if case["dist"] == "words":
        letters, lens = vocabulary
        # words by Zipf's law, a space after each
        weight = 1.0 / (torch.arange(VOCABULARY, device="cuda") + 2.7)
        lens_d = torch.from_numpy(lens).cuda()
        start = torch.cumsum(lens_d, 0) - lens_d
        letters_d = torch.from_numpy(letters).cuda()
        at = 0
        while at < n:
            ids = torch.multinomial(weight, 200_000, replacement=True, generator=gen)
            ln = lens_d[ids] + 1
            begin = torch.cumsum(ln, 0) - ln
            word = torch.repeat_interleave(torch.arange(len(ids), device="cuda"), ln)
            j = torch.arange(len(word), device="cuda") - begin[word]
            inside = j < lens_d[ids[word]]
            src = (start[ids[word]] + j).clamp_(max=len(letters) - 1)
            part = torch.where(inside, letters_d[src], torch.full_like(letters_d[src], 32))
            m = min(n - at, len(part))
            out[at:at + m] = part[:m]
            at += m
        return
    for a in range(0, n, 64 * MiB):
        m = min(64 * MiB, n - a)
        part = out[a:a + m]
        if case["dist"] == "uniform":
            part.random_(0, 256, generator=gen)
        elif case["dist"] == "mix":
            part.random_(0x20, 0x7F, generator=gen)
            other = torch.empty_like(part).random_(0, 256, generator=gen)
            pick = torch.empty_like(part).random_(0, 10, generator=gen)
            part.copy_(torch.where(pick < 7, part, other))
        else:
            part.random_(0, 4, generator=gen)
            part.copy_(torch.from_numpy(np.frombuffer(b"ACGT", dtype=np.uint8).copy()).cuda()[part.int()])


def _plant(case, n, pats, rng, out):
    """Write copies of patterns, one in each of n // gap stretches of `gap`
    bytes at a random place, so that no two overlap (in a batch some cross the
    end of a text and are no match)."""
    gap = case["gap"]
    slots = n // gap
    lens = np.diff(pats.offsets).astype(np.int64)
    data = torch.from_numpy(pats.data.copy()).cuda()
    step = 1 << 17
    for a in range(0, slots, step):
        m = min(step, slots - a)
        ids = rng.integers(0, case["k"], m)
        ln = lens[ids]
        pos = (a + np.arange(m)) * gap + rng.integers(0, gap - ln + 1)
        ln_d = torch.from_numpy(ln).cuda()
        begin = torch.cumsum(ln_d, 0) - ln_d
        copy = torch.repeat_interleave(torch.arange(m, device="cuda"), ln_d)
        j = torch.arange(len(copy), device="cuda") - begin[copy]
        src = torch.from_numpy(pats.offsets[ids].astype(np.int64)).cuda()[copy] + j
        out[torch.from_numpy(pos).cuda()[copy] + j] = data[src]


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    vocabulary = _vocabulary(rng) if case["dist"] == "words" else None
    pats = _patterns(case, rng, vocabulary)
    n = _total(case)
    shift = case.get("shift", 0)
    buffer = torch.empty(n + shift, dtype=torch.uint8, device="cuda")
    text = buffer[shift:]
    _text(case, n, gen, vocabulary, text)
    _plant(case, n, pats, rng, text)
    s = types.SimpleNamespace(case=case, n=n, trie=pf.Trie(pats), text=text)
    s.capacity = 1024 + 2 * int(_expected(case))
    if case["call"] == "serve":
        lens = _lengths(case)
        host = text.cpu().pin_memory()
        ends = np.cumsum(lens)
        s.texts = [host[e - ln:e].numpy() for e, ln in zip(ends.tolist(), lens.tolist())]
        s.text = None
        budget = 64 * MiB
        arena = torch.empty(budget + 16 * MiB, dtype=torch.uint8, device="cuda")
        s.server = pf.Server(s.trie, arena, budget, 64, torch.cuda.Stream(), torch.cuda.Stream())
        # where the caller gathers its requests' records
        s.room = 64 + 2 * lens // case["gap"]
        s.found = np.zeros((int(s.room.sum()), RECORD // 8), dtype=np.int64)
        return s
    s.ws = pf.Workspace()
    s.out = torch.zeros(s.capacity * RECORD, dtype=torch.uint8, device="cuda")
    s.count = torch.zeros(1, dtype=torch.int64, device="cuda")
    s.counts = torch.zeros(n, dtype=torch.int32, device="cuda") if case.get("counts") else None
    if "small" in case:
        offsets = np.zeros(len(_lengths(case)) + 1, dtype=np.int64)
        offsets[1:] = np.cumsum(_lengths(case))
        s.offsets = torch.from_numpy(offsets).cuda()
        s.n_texts = len(offsets) - 1
        if case["call"] == "graph":
            torch.cuda.synchronize()
            s.graph = pf.Graph(s.trie, None, s.text, s.offsets, s.n_texts, n, s.out, s.capacity, s.count)
    return s


# --------------------------------------------------------------------- pass


def run(s):
    call = s.case["call"]
    if call == "scan":
        pf.pfac_scan(s.trie, s.ws, s.text, s.n, s.out, s.capacity, s.count, s.counts)
        return {"matches": s.out, "count": s.count, "counts": s.counts}
    if call == "scan_sync":
        rc, found = pf.pfac_scan_sync(s.trie, s.ws, s.text, s.n, s.out, s.capacity, s.counts)
        return {"matches": s.out, "count": found, "rc": rc}
    if call == "scan_noalloc":
        pf.pfac_scan_noalloc(s.trie, s.text, s.n, s.out, s.capacity, s.count, s.counts)
        return {"matches": s.out, "count": s.count}
    if call == "batch":
        pf.pfac_scan_batch(s.trie, s.ws, s.text, s.offsets, s.n_texts, s.n, s.out, s.capacity, s.count)
        return {"matches": s.out, "count": s.count}
    if call == "graph":
        s.graph.launch()
        return {"matches": s.out, "count": s.count}
    ids = [s.server.submit(t) for t in s.texts]
    found, at = [], 0
    for i, room in zip(ids, s.room.tolist()):
        m, _ = s.server.wait(i, capacity=room)
        s.found[at:at + len(m)] = m.view(np.int64).reshape(-1, RECORD // 8)
        found.append(len(m))
        at += room
    return {"matches": s.found, "found": np.array(found)}


def work(case):
    """Each text byte read once, each match record (and count) written once;
    a batch's offsets are read too."""
    n = _total(case)
    b = n + RECORD * _expected(case)
    if case.get("counts"):
        b += 4 * n
    if "small" in case:
        b += 8 * (case["small"] + case["large"] + 1)
    return {"bytes": int(b), "flops": 0}
