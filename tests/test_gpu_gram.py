"""The gram kernel (launches whose kernel the library chooses, patterns of
four bytes or more; grams of up to 16 symbols over four) against the oracle,
record by record: each distance of test positions, texts at odd addresses whose
ends fall inside a chunk, starts at every offset around a unit's edge, batches
of tiny and empty texts, matches past the LDS list of a unit and past its list
in global memory."""

import numpy as np
import pytest

import oracle
import paper_1702_03657_amd as pf
from tests.gpu_util import assert_same, gpu_scan, gpu_scan_batch, say

pytestmark = pytest.mark.gpu

MiB = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pf.load()


def _patterns(rng, k, lo, hi, alphabet):
    return [bytes(rng.choice(alphabet, int(rng.integers(lo, hi + 1))).astype(np.uint8)) for _ in range(k)]


BYTES = np.arange(256)
LOWER = np.arange(97, 123)


# shortest pattern 4 tests every position, 5 and 6 every second, 7 and more
# every fourth; units of one chunk and of up to 64, with the bitmap in LDS and
# read from global memory (up to 2,560 chunks when it is past 16 KiB)
@pytest.mark.parametrize("lo,alphabet,n,pad", [
    (4, BYTES, 1, 0), (4, BYTES, 64, 3), (5, BYTES, 1023, 1), (7, BYTES, 1025, 15), (8, BYTES, 16 * 1024 + 9, 5),
    (8, BYTES, 1280 * 1024 - 5, 5), (6, BYTES, 1280 * 1024 + 1, 0), (8, BYTES, 2560 * 1024, 0),
    (7, BYTES, 2560 * 1024 + 1, 0), (5, BYTES, 2560 * 1024 + 16, 7), (4, LOWER, 300_001, 11), (8, BYTES, 5_000_011, 3),
    (4, BYTES, 8 * MiB + 1, 0), (5, BYTES, 8 * MiB + 1023, 1), (6, BYTES, 9 * MiB + 7, 13),
    (7, BYTES, 8 * MiB, 15), (8, BYTES, 40 * MiB + 4093, 3), (4, LOWER, 8 * MiB + 77, 2), (7, LOWER, 9 * MiB, 9),
])
def test_one_text(lo, alphabet, n, pad):
    rng = np.random.default_rng(lo * 100 + pad)
    pats = _patterns(rng, 1500, lo, lo + 24, alphabet)
    text = rng.choice(alphabet, n).astype(np.uint8)
    for q in range(0 if n < 64 else max(n // 3000, 8)):  # whole copies and copies cut short
        p = np.frombuffer(pats[int(rng.integers(0, len(pats)))], dtype=np.uint8)
        at = int(rng.integers(0, n - p.size + 1))
        m = p.size if q % 4 else int(rng.integers(1, p.size + 1))
        text[at:at + m] = p[:m]
    if n >= 64:  # both ends of the text
        first, last = (np.frombuffer(p, dtype=np.uint8) for p in pats[:2])
        text[:first.size] = first
        text[n - last.size:] = last
    for e in range(16 if n > 8 * MiB else 1, 4096, 16 if n > 8 * MiB else 3):  # starts around the edges of units
        p = np.frombuffer(pats[e % len(pats)], dtype=np.uint8)
        at = e * 1024 - pad + e // 3 % 8 - 4
        if at + p.size <= n - 40:
            text[at:at + p.size] = p
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram lo={lo} n={n} pad={pad}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=pad)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


@pytest.mark.parametrize("total", [30_000, 3 * MiB, 8 * MiB + 50])
@pytest.mark.parametrize("lo,most,graph", [(4, 40, 0), (5, 300, 3), (8, 3000, 0), (9, 70_000, 2)])
def test_batch(lo, most, graph, total):
    rng = np.random.default_rng(lo)
    pats = _patterns(rng, 900, lo, lo + 20, np.arange(32, 48))
    lens = []
    while sum(lens) < total + 100:
        lens += rng.integers(0, most, 4000).tolist() + [0, 0, 1, 2, 3]
    lens = lens[:next(i for i, t in enumerate(np.cumsum(lens)) if t > total) + 1]
    offs = np.zeros(len(lens) + 1, dtype=np.uint64)
    offs[1:] = np.cumsum(lens)
    n = int(offs[-1])
    text = rng.choice(np.arange(32, 48), n).astype(np.uint8)
    for _ in range(n // 300 if n < MiB else n // 1000):
        p = np.frombuffer(pats[int(rng.integers(0, len(pats)))], dtype=np.uint8)
        at = int(rng.integers(0, n - p.size))
        text[at:at + p.size] = p
    want = oracle.bucketed(text, pats, offsets=offs, threads=8)
    say(f"gram batch lo={lo}: {len(lens)} texts, {n} bytes, {want.n} matches")
    got, cnt = gpu_scan_batch(pf.Trie(pats), text, offs, pad_front=lo, graph_replays=graph)
    assert cnt == want.n
    for g in (got if graph else [got]):
        assert_same(g, want, with_text=True)


@pytest.mark.parametrize("lo,n", [(4, 8 * MiB + 333), (5, 8 * MiB + 333), (7, 8 * MiB + 333), (5, MiB + 3),
                                  (7, 4 * MiB + 1)])
@pytest.mark.parametrize("density", ["spill", "redo", "nested"])
def test_dense_matches(lo, n, density):
    """Stretches of many matches in units that hold few elsewhere."""
    rng = np.random.default_rng(lo)
    text = rng.integers(0, 200, n).astype(np.uint8)
    if density == "nested":
        pats = [b"\xff" * m for m in range(lo, lo + 9)] * 2 + [b"\xfe" * lo + b"\xff"]
        for at in (5000, n // 2 + 1, n - 3000):
            text[at:at + 2500] = 0xff
    else:
        pats = _patterns(rng, 40, lo, lo + 3, np.arange(200, 256))
        step = 40 if density == "spill" else 11
        for lo_at in (0, n // 2 + 1):  # past 64 matches a unit, past 32 a KiB
            for q in range(3000):
                p = np.frombuffer(pats[q % len(pats)], dtype=np.uint8)
                at = lo_at + q * step
                text[at:at + p.size] = p
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram dense {density} lo={lo}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


@pytest.mark.parametrize("n", [100_003, 3 * MiB + 5, 9 * MiB])
@pytest.mark.parametrize("lo,dup", [(4, False), (5, True), (7, False)])
def test_nested_words(lo, dup, n):
    """Words that are prefixes of others or equal, in text made of them: grams
    of one trie node with more than one string below it (walked from that
    node), of several nodes, and lists of several ids."""
    rng = np.random.default_rng(n + lo)
    stems = _patterns(rng, 120, lo, lo + 2, LOWER)
    pats = stems + [s + bytes(rng.choice(LOWER, int(rng.integers(1, 6))).astype(np.uint8)) for s in stems for _ in range(2)]
    # the same tails behind other heads: one gram at several nodes
    pats += [bytes(rng.choice(LOWER, 2).astype(np.uint8)) + s for s in stems[:40] if lo >= 5]
    if dup:
        pats += pats[::3]
    words = [pats[int(i)] + bytes(rng.choice(LOWER, int(j)).astype(np.uint8))
             for i, j in zip(rng.integers(0, len(pats), n // 60), rng.integers(0, 60, n // 60))]
    text = np.frombuffer(b"".join(words), dtype=np.uint8)[:n]
    text = np.concatenate([text, rng.choice(LOWER, n - text.size).astype(np.uint8)])
    text[-lo:] = np.frombuffer(stems[0][:lo], dtype=np.uint8)
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram words lo={lo} dup={dup} n={n}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=n % 16)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


# four symbols: grams of up to 16 of them.  Short patterns (grams of 4 to 13
# symbols, every position, every second or every fourth), long ones (16, and from
# 19 on runs of four in large sets), sets that fill the bitmap; alphabets of two and three symbols, bytes that share the
# symbols' bits (upper case, N) in runs and alone, both ends of the text, starts
# around the edges of units, runs of one symbol
@pytest.mark.parametrize("alphabet", [b"acgt", b"ACT", b"01"])
@pytest.mark.parametrize("lo,k,n,pad", [
    (9, 500, 70, 3), (9, 60, 1023, 1), (9, 500, 1025, 15), (10, 300, 300_001, 11), (12, 500, 2560 * 1024, 7),
    (20, 1000, 2560 * 1024 + 1, 0), (6, 20, 3 * MiB, 5), (9, 500, 8 * MiB + 1, 2), (13, 400, 9 * MiB, 13),
    (19, 40_000, 5 * MiB + 3, 4), (18, 40_000, 5 * MiB, 8), (20, 40_000, 9 * MiB + 1023, 9),
    (24, 100_000, 20 * MiB + 5, 1),
])
def test_symbols(lo, k, n, pad, alphabet):
    rng = np.random.default_rng(lo + k + len(alphabet))
    a = np.frombuffer(alphabet, dtype=np.uint8)
    if len(alphabet) == 2:
        lo *= 2
    pats = _patterns(rng, k, lo, lo + 12, a)
    text = rng.choice(a, n).astype(np.uint8)
    if n > MiB:
        text[n // 3:n // 3 + 9000] = ord("N")
        text[n // 5:n // 5 + 40_000] ^= 0x20
        other = rng.integers(0, n, n // 500)
        text[other] = rng.integers(0, 256, other.size)
        pats += [alphabet[:1] * lo, alphabet[1:2] * (lo + 3), alphabet[-1:] * 40]
        text[n // 2:n // 2 + 700] = a[0]
    for q in range(max(n // 3000, 4)):
        p = np.frombuffer(pats[int(rng.integers(0, len(pats)))], dtype=np.uint8)
        at = int(rng.integers(0, n - p.size + 1))
        m = p.size if q % 4 else int(rng.integers(1, p.size + 1))
        text[at:at + m] = p[:m]
    for e in range(1, n // 1024, 16 if n > 8 * MiB else 3):
        p = np.frombuffer(pats[e % len(pats)], dtype=np.uint8)
        at = e * 1024 - pad + e // 3 % 24 - 20
        if at >= 0 and at + p.size <= n - 40:
            text[at:at + p.size] = p
    first, last = (np.frombuffer(p, dtype=np.uint8) for p in pats[:2])
    text[:first.size] = first
    text[n - last.size:] = last
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram symbols {alphabet} lo={lo} k={k} n={n}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=pad)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))


@pytest.mark.parametrize("lo,k,most", [(9, 300, 60), (12, 500, 2000), (20, 5000, 40_000), (20, 60_000, 900)])
def test_symbols_batch(lo, k, most):
    rng = np.random.default_rng(lo)
    a = np.frombuffer(b"acgt", dtype=np.uint8)
    pats = _patterns(rng, k, lo, lo + 10, a)
    lens = rng.integers(0, most, 6 * MiB // most).tolist() + [0, 0, 1, lo]
    offs = np.zeros(len(lens) + 1, dtype=np.uint64)
    offs[1:] = np.cumsum(lens)
    n = int(offs[-1])
    text = rng.choice(a, n).astype(np.uint8)
    for _ in range(n // 800):
        p = np.frombuffer(pats[int(rng.integers(0, len(pats)))], dtype=np.uint8)
        at = int(rng.integers(0, n - p.size))
        text[at:at + p.size] = p
    want = oracle.bucketed(text, pats, offsets=offs, threads=8)
    say(f"gram symbols batch lo={lo}: {len(lens)} texts, {n} bytes, {want.n} matches")
    got, cnt = gpu_scan_batch(pf.Trie(pats), text, offs, pad_front=lo)
    assert cnt == want.n
    assert_same(got, want, with_text=True)
