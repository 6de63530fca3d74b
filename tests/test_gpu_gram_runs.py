"""Texts that repeat themselves (padding, blank space, tables, unknown bases)
against sets that hold what is repeated: record by record against the oracle,
and the time of a scan, which must not follow the length of the runs when no
pattern can start in them."""

import numpy as np
import pytest

import oracle
import paper_1702_03657_amd as pf
from tests.gpu_util import assert_same, gpu_scan, say

pytestmark = pytest.mark.gpu

MiB = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pf.load()


FILLS = [b"\0", b" ", b"\xff", b"\0\xff", b"\x01\0\0\0", b"\xef\xbe\xad\xde", b"\0\x01\x02\x03\x04\x05\x06\x07"]


def _fill_patterns(rng, lo):
    """Patterns that begin in a run, end in one, lie in one and only touch one,
    at every phase of it."""
    pats = []
    for f in FILLS:
        for phase in range(len(f)):
            run = (f[phase:] + f[:phase]) * 12
            for head in range(5):  # heads that go on with the run and heads that do not
                h = bytes(rng.integers(65, 91, head).astype(np.uint8))
                for m in {4, 5, 6, 7, 9, 12}:
                    if head + m >= lo:
                        pats.append(h + run[:m])
                    pats.append((h + run[:m] + bytes(rng.integers(97, 123, lo).astype(np.uint8)))[:max(lo, head + m + 2)])
    return list(dict.fromkeys(pats))


# 150 more patterns: small bitmap, long lists; 20,000: bitmap in LDS or, up to
# 2.5 MiB, read from L2
@pytest.mark.parametrize("n,pad", [(70_000, 1), (1 * MiB + 3, 6), (5 * MiB, 15)])
@pytest.mark.parametrize("more", [150, 20_000])
@pytest.mark.parametrize("lo", [4, 5, 8])
def test_runs(lo, more, n, pad):
    rng = np.random.default_rng(lo * more + n)
    fills = _fill_patterns(rng, lo)
    pats = fills + [rng.integers(0, 256, int(rng.integers(lo, 24)), dtype=np.uint8).tobytes() for _ in range(more)]
    text = rng.integers(0, 256, n, dtype=np.uint8)
    at = 0
    while at < n - 5000:
        f = FILLS[int(rng.integers(0, len(FILLS)))]
        m = int(rng.choice([3, 4, 5, 7, 8, 9, 17, 40, 70, 1100, 2500], p=[.12, .12, .12, .12, .12, .1, .1, .08, .06, .04, .02]))
        at += int(rng.integers(1, 900 if n > MiB else 300))
        text[at:at + m] = np.resize(np.frombuffer(f, dtype=np.uint8), m)
        if rng.random() < 0.7:  # a pattern across the run's first or last byte, or inside it
            p = np.frombuffer(fills[int(rng.integers(0, len(fills)))], dtype=np.uint8)
            q = max(0, at + int(rng.choice([-4, -3, -2, -1, 0, 1, 5, m - 9, m - 6, m - 4])))
            text[q:q + p.size] = p
        at += m
    text[-40:] = 0
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram runs lo={lo} more={more} n={n}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=pad, capacity=want.n)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


@pytest.mark.parametrize("lo", [5, 8])
@pytest.mark.parametrize("more", [150, 20_000])
@pytest.mark.parametrize("kib", [600, 9000])
def test_runs_from_a_chunk_s_first_byte(lo, more, kib):
    """Runs that begin where a KiB of the text's frame does, behind the first
    bytes of a pattern that goes on with them, after runs of other bytes: what
    lies before the chunk is not what a run inside it suggests."""
    rng = np.random.default_rng(lo + more)
    fills = [b"\xff", b"\0", b"\0\0\xff\xff", b"\xff\xff\0\0", b"\0\xff", b"\x01\x02\x03\x04\x05\x06\x07\x08"]
    heads = [b"M", b"MZ", b"M\0Z"]
    # a pattern for each head and phase of a fill, none that begins in one
    pats = [h + ((f[q:] + f[:q]) * 8)[:m] for f in fills for h in heads for q in range(len(f)) for m in (lo, lo + 1, 20)]
    pats += [bytes(rng.integers(1, 255, 1, dtype=np.uint8)) + rng.integers(0, 256, int(rng.integers(lo, 24)), dtype=np.uint8).tobytes()
             for _ in range(more)]
    pad = 5
    n = kib * 1024 + 77
    text = rng.integers(0, 256, n, dtype=np.uint8)
    for c in range(2, kib - 10):
        at = c * 1024 - pad
        f = fills[c % len(fills)]
        q = int(rng.integers(0, len(f)))
        h = np.frombuffer(heads[c // len(fills) % len(heads)] if c % 4 else f[-1:], dtype=np.uint8)
        text[at:at + 200] = np.resize(np.frombuffer(f[q:] + f[:q], dtype=np.uint8), 200)
        text[at - h.size:at] = h
        # another run before, so that a wave has seen one
        g = np.frombuffer(fills[(c + 1) % len(fills)], dtype=np.uint8)
        text[at - 300:at - 100] = np.resize(g, 200)
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram runs at chunks lo={lo} more={more} kib={kib}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=pad, capacity=want.n)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


@pytest.mark.parametrize("lo,hi,k", [(9, 14, 300), (13, 16, 3000), (20, 32, 20_000)])
def test_symbol_runs(lo, hi, k):
    rng = np.random.default_rng(lo)
    a = np.frombuffer(b"ACGT", dtype=np.uint8)
    n = 4 * MiB + 11
    pats = [bytes(rng.choice(a, int(m))) for m in rng.integers(lo, hi + 1, k)]
    pats += [b"G" * lo, b"A" * (lo + 2), b"C" + b"G" * lo, b"G" * lo + b"TC", b"AC" * lo]
    text = rng.choice(a, n)
    for at in range(3000, n - 9000, 60_000):
        c = [b"N", b"G", b"n", b"A", b"\n"][at // 60_000 % 5]
        m = int(rng.integers(10, 5000))
        text[at:at + m] = c[0]
        for q in (at - 1, at + m - 1, at + m // 2):  # a pattern at each end and in the middle
            p = np.frombuffer(pats[-int(rng.integers(1, 6))], dtype=np.uint8)
            text[q:q + p.size] = p
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram symbol runs lo={lo}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=3, capacity=want.n)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


def _time(trie, text):
    """Microseconds of a scan, the least of several runs of five."""
    import torch
    dev = torch.from_numpy(text).cuda()
    ws, n, cap = pf.Workspace(), text.size, 1 << 16
    out = torch.empty(cap * 16, dtype=torch.uint8, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    best = 1e9
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(9):
        a.record()
        for _ in range(5):
            pf.pfac_scan(trie, ws, dev, n, out, cap, cnt)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 200)
    return best, int(cnt.item())


# Where every test of a run was checked, a tenth of the text in runs took 3 (4
# KiB of zeros) to 13 times (N) the time of the text without them.
@pytest.mark.parametrize("fill,size,lo", [(b"\0", 1 << 16, 8), (b"\0", 1 << 12, 8), (b"\0", 1 << 16, 5),
                                          (b"\xff\0", 1 << 16, 8), (b"N", 1 << 20, 20), (b"N", 1 << 20, 9)])
def test_time_of_runs(fill, size, lo):
    rng = np.random.default_rng(size + lo)
    n = 64 * MiB
    if fill == b"N":
        a = np.frombuffer(b"ACGT", dtype=np.uint8)
        pats = [bytes(rng.choice(a, int(m))) for m in rng.integers(lo, lo + 6, 5000 if lo > 16 else 500)] + [b"G" * lo]
        text = rng.choice(a, n)
    else:
        pats = [bytearray(rng.integers(1, 255, int(m), dtype=np.uint8).tobytes()) for m in rng.integers(lo, 64, 8000)]
        for i, p in enumerate(pats[:80]):
            o = 1 + i % 3 if lo >= 7 else 1
            p[o:o + 4] = (fill * 4)[:4]
        pats = [bytes(p) for p in pats]
        text = rng.integers(0, 256, n, dtype=np.uint8)
    trie = pf.Trie(pats)
    plain, found = _time(trie, text)
    for at in rng.integers(0, n - size, max(n // 10 // size, 1)):
        text[at:at + size] = np.resize(np.frombuffer(fill, dtype=np.uint8), size)
    runs, found_runs = _time(trie, text)
    say(f"runs of {fill!r} x {size}, lo {lo}: {plain:.1f} us without, {runs:.1f} with ({found}, {found_runs} matches)")
    assert runs < 1.5 * plain
