"""The launches whose kernel the library chooses, through every entry point and
against the oracle: each form of the gram kernel (bytes and symbols, distance of
tests, bitmap in LDS or read from L2; the library is asked that it is the one),
counts beyond the capacity, texts of every length around the patterns' and at
every address, random sets, requests through the server, and scans without
allocation on both sides of what the scratch holds."""

import numpy as np
import pytest

import oracle
import paper_1702_03657_amd as pf
from tests.gpu_util import assert_same, gpu_scan, gpu_scan_batch, say

pytestmark = pytest.mark.gpu

KiB, MiB = 1 << 10, 1 << 20
BYTES = np.arange(256, dtype=np.uint8)
DNA = np.frombuffer(b"ACGT", dtype=np.uint8)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    pf.load()


def _patterns(rng, alphabet, k, lo, hi):
    return [rng.choice(alphabet, int(m)).tobytes() for m in rng.integers(lo, hi + 1, k)]


def _text(rng, alphabet, n, pats, gap=300):
    """Random text with a pattern every `gap` bytes and two dense stretches."""
    text = rng.choice(alphabet, n)

    def put(at):
        p = np.frombuffer(pats[int(rng.integers(0, len(pats)))], dtype=np.uint8)
        m = min(p.size, n - at)
        text[at:at + m] = p[:m]

    for at in range(0, n, gap):
        put(at + int(rng.integers(0, gap)) if at + gap < n else at)
    for at in range(n // 3, min(n, n // 3 + 20_000), 40):
        put(at)
    for at in range(n // 2, min(n, n // 2 + 20_000), 13):
        put(at)
    return text


FORMS = [  # alphabet, lo, hi, k, bytes, (step, symbols, runs, bitmap in LDS)
    (BYTES, 8, 24, 300, 600_000, (4, 0, 0, 1)), (BYTES, 8, 24, 6000, 600_000, (4, 0, 0, 0)),
    (BYTES, 8, 24, 6000, 4 * MiB, (4, 0, 0, 1)), (BYTES, 5, 24, 6000, 600_000, (2, 0, 0, 0)),
    (BYTES, 6, 24, 6000, 4 * MiB, (2, 0, 0, 1)), (BYTES, 4, 24, 9000, 600_000, (1, 0, 0, 0)),
    (BYTES, 4, 24, 9000, 4 * MiB, (1, 0, 0, 1)), (DNA, 20, 32, 4000, 900_000, (4, 16, 0, 0)),
    (DNA, 20, 32, 4000, 4 * MiB, (4, 16, 0, 1)), (DNA, 12, 16, 4000, 900_000, (2, 11, 0, 0)),
    (DNA, 12, 16, 4000, 4 * MiB, (2, 11, 0, 1)), (DNA, 12, 16, 20_000, 900_000, (1, 12, 0, 0)),
    (DNA, 12, 16, 20_000, 4 * MiB, (1, 12, 0, 1)), (DNA, 20, 32, 60_000, 900_000, (1, 16, 1, 0)),
    (DNA, 20, 32, 60_000, 4 * MiB, (1, 16, 1, 1)),
]


@pytest.mark.parametrize("alphabet,lo,hi,k,n,form", FORMS, ids=["-".join(map(str, f[5] + (f[4],))) for f in FORMS])
def test_every_form_and_entry_point(alphabet, lo, hi, k, n, form):
    import torch
    rng = np.random.default_rng(k + n)
    pats = _patterns(rng, alphabet, k, lo, hi)
    n += 7
    text = _text(rng, alphabet, n, pats)
    trie = pf.Trie(pats)
    told = trie.launch_gram(n)
    assert (told["step"], told["symbols"], told["runs"], told["bitmap_in_lds"]) == form
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram form {told}: {want.n} matches")
    got, counts = gpu_scan(trie, text, pad_front=9, capacity=want.n)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))

    # less room than matches: the count is exact, and the workspace serves on
    ws = pf.Workspace()
    dev = torch.from_numpy(text).cuda()
    for cap in (0, 100, want.n // 2):
        out = torch.empty(max(cap, 1) * 16, dtype=torch.uint8, device="cuda")
        rc, cnt = pf.pfac_scan_sync(trie, ws, dev, n, out if cap else None, cap)
        assert rc == pf.PFAC_ETRUNC and cnt == want.n
    got, _ = gpu_scan(trie, text, ws=ws, counts=False, capacity=want.n)
    assert_same(got, want)

    # without allocation, twice
    out = torch.empty(want.n * 16, dtype=torch.uint8, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    for _ in range(2):
        out.fill_(0xAB)
        pf.pfac_scan_noalloc(trie, dev, n, out, want.n, cnt)
        torch.cuda.synchronize()
        assert int(cnt.item()) == want.n
        assert_same(pf.matches_to_numpy(out, want.n), want)

    # as a batch, one text after another, and replayed
    lens = np.concatenate([rng.integers(0, 60, 400), rng.integers(0, 3000, 200), [0, 0, lo - 1, lo]])
    lens = lens[np.cumsum(lens) < n]
    offs = np.zeros(len(lens) + 2, dtype=np.uint64)
    offs[1:-1] = np.cumsum(lens)
    offs[-1] = n
    want = oracle.bucketed(text, pats, offsets=offs, threads=8)
    got, cnt_b = gpu_scan_batch(trie, text, offs, pad_front=3)
    assert_same(got, want, with_text=True)
    if n < MiB:
        got, cnt_b = gpu_scan_batch(trie, text, offs, plain=True)
        assert_same(got, want, with_text=True)
    d_offs = torch.from_numpy(offs.view(np.int64)).cuda()
    out = torch.empty(want.n * 16, dtype=torch.uint8, device="cuda")
    graph = pf.Graph(trie, None, dev, d_offs, len(offs) - 1, n, out, want.n, cnt)
    for _ in range(4):  # eager scans and synchronisations between the replays
        out.fill_(0xAB)
        graph.launch()
        torch.cuda.synchronize()
        assert int(cnt.item()) == want.n
        assert_same(pf.matches_to_numpy(out, want.n), want, with_text=True)
        one, _ = gpu_scan(trie, text[:5000], ws=ws, counts=False)
        assert_same(one, oracle.bucketed(text[:5000], pats, threads=8))
    graph.close()


@pytest.mark.parametrize("lo", [4, 5, 8])
def test_texts_around_the_patterns_lengths(lo):
    rng = np.random.default_rng(lo)
    pats = _patterns(rng, BYTES, 50, lo, 40) + [b"tail!tail!"[:max(lo, 5)]]
    trie = pf.Trie(pats)
    assert trie.launch_gram(1)["step"] and trie.launch_gram(0)["step"]
    ws = pf.Workspace()
    for n in list(range(0, 45)) + [1023, 1024, 1025, 2047, 2048]:
        pad = n % 16
        text = rng.choice(BYTES, n)
        p = np.frombuffer(pats[n % len(pats)], dtype=np.uint8)
        if p.size <= n:  # a pattern at the end, another at the start where both fit
            text[n - p.size:] = p
            q = np.frombuffer(pats[(n + 7) % len(pats)], dtype=np.uint8)
            if q.size + p.size <= n:
                text[:q.size] = q
        want = oracle.brute(text, pats)
        got, counts = gpu_scan(trie, text, ws=ws, pad_front=pad)
        assert_same(got, want)
        if n:
            assert np.array_equal(counts, oracle.counts(n, want))


@pytest.mark.parametrize("case", ["duplicates", "nested", "long", "dense_candidates", "one_pattern"])
def test_special_sets(case):
    rng = np.random.default_rng(11)
    if case == "duplicates":
        pats = [b"abab", b"xyzxyz", b"abab", b"babab", b"abab", b"ababxyz", b"xyzxyz"]
        text = rng.choice(np.frombuffer(b"abxyz", dtype=np.uint8), 30_000)
    elif case == "nested":
        pats = [b"a" * d for d in range(4, 40)] + [b"q!" * 6]
        text = np.frombuffer(b"a" * 20_000 + b"b" + b"a" * 5000 + b"q!" * 30, dtype=np.uint8).copy()
    elif case == "long":  # past 65,535 bytes: no record holds the length
        base = rng.integers(0, 100, 200_000, dtype=np.uint8)
        pats = [base[:70_000].tobytes(), base[:70_000].tobytes() + b"\xff", base[1000:66_535].tobytes(),
                base[5:66_000].tobytes(), base[40:48].tobytes()]
        text = np.concatenate([base, base[:150_000]])
    elif case == "dense_candidates":
        pats = [b"aaaab", b"aaaxb", b"aaaabx", b"baaaa!"]
        text = np.frombuffer((b"a" * 3000 + b"b") * 12, dtype=np.uint8).copy()
    else:
        pats = [b"needle"]
        text = np.frombuffer(b"hay" * 5000 + b"needle" + b"ne" * 300 + b"needlneedle", dtype=np.uint8).copy()
    trie = pf.Trie(pats)
    say(f"gram special {case}: {trie.launch_gram(text.size)}")
    want = oracle.bucketed(text, pats, threads=8)
    got, counts = gpu_scan(trie, text, pad_front=5)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(text.size, want))


@pytest.mark.parametrize("seed", range(30))
def test_random_sets(seed):
    """Sets of any alphabet whose shortest pattern has four bytes or more, in
    texts and batches of any size, with the tuning the build chose."""
    rng = np.random.default_rng(1000 + seed)
    alphabet = [BYTES, np.arange(32, 127, dtype=np.uint8), np.arange(97, 123, dtype=np.uint8), DNA,
                np.frombuffer(b"01", dtype=np.uint8), np.arange(0, 12, dtype=np.uint8)][seed % 6]
    lo = int(rng.integers(4, 10)) * (3 if alphabet.size == 2 else 1)
    k = int(np.exp(rng.uniform(0, np.log(4000))))
    pats = _patterns(rng, alphabet, k, lo, lo + int(rng.integers(0, 40)))
    pats += [p[:max(lo, len(p) // 2)] for p in pats[::5]] + pats[::9]
    trie = pf.Trie(pats)
    for n in (int(np.exp(rng.uniform(3, np.log(300_000)))), int(rng.integers(1 << 20, 5 << 20))):
        text = _text(rng, alphabet, n, pats, gap=int(rng.integers(60, 3000)))
        want = oracle.bucketed(text, pats, threads=8)
        say(f"gram random {seed}: k={k} lo={lo} n={n} {trie.launch_gram(n)['step']}: {want.n} matches")
        got, counts = gpu_scan(trie, text, pad_front=int(rng.integers(0, 16)))
        assert_same(got, want)
        assert np.array_equal(counts, oracle.counts(n, want))
        cuts = np.sort(rng.integers(0, n + 1, int(rng.integers(1, 300))))
        offs = np.concatenate([[0], cuts, [n]]).astype(np.uint64)
        want = oracle.bucketed(text, pats, offsets=offs, threads=8)
        got, _ = gpu_scan_batch(trie, text, offs, pad_front=int(rng.integers(0, 16)))
        assert_same(got, want, with_text=True)


@pytest.mark.parametrize("alphabet", ["bytes", "words"])
@pytest.mark.parametrize("room", [16 * MiB, 24 * KiB])
def test_server(alphabet, room):
    """Requests through the server; with little room for records, batches
    overflow and each of their requests is scanned alone."""
    import torch
    rng = np.random.default_rng(room)
    a = BYTES if alphabet == "bytes" else np.arange(97, 123, dtype=np.uint8)
    pats = _patterns(rng, a, 2000, 6, 40)
    trie = pf.Trie(pats)
    assert trie.launch_gram(MiB)["step"]
    texts = [_text(rng, a, int(n), pats) for n in np.exp(rng.uniform(np.log(500), np.log(400_000), 24))]
    budget = 2 * MiB
    arena = torch.empty(budget + 2 * room, dtype=torch.uint8, device="cuda")
    server = pf.Server(trie, arena, budget, 8, torch.cuda.Stream(), torch.cuda.Stream())
    ids = [server.submit(t) for t in texts]
    for t, i in zip(texts, ids):
        got, _ = server.wait(i, capacity=1 << 16)
        assert_same(got, oracle.bucketed(t, pats, threads=8))
    server.close()


def test_noalloc_on_both_sides_of_the_scratch():
    """A capacity that leaves no room for the list area in the 64 MiB, and one
    that does."""
    import torch
    rng = np.random.default_rng(2)
    pats = _patterns(rng, BYTES, 3000, 8, 40)
    n = 7 * MiB + 5
    text = _text(rng, BYTES, n, pats, gap=2000)
    want = oracle.bucketed(text, pats, threads=8)
    trie = pf.Trie(pats)
    dev = torch.from_numpy(text).cuda()
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    for cap in (want.n, (62 * MiB) // 16):
        out = torch.empty(cap * 16, dtype=torch.uint8, device="cuda")
        counts = torch.full((n,), 7, dtype=torch.int32, device="cuda")
        for _ in range(2):
            out.fill_(0xAB)
            pf.pfac_scan_noalloc(trie, dev, n, out, cap, cnt, counts)
            torch.cuda.synchronize()
            assert int(cnt.item()) == want.n
            assert_same(pf.matches_to_numpy(out, want.n), want)
            assert np.array_equal(counts.cpu().numpy().view(np.uint32), oracle.counts(n, want))


@pytest.mark.parametrize("noalloc", [False, True])
def test_scans_captured_by_the_caller(noalloc):
    """A scan captured on the caller's stream as a workspace's first one, then
    replayed, with eager scans of other sizes on the same workspace between."""
    import torch
    rng = np.random.default_rng(5)
    pats = _patterns(rng, BYTES, 500, 5, 30)
    trie = pf.Trie(pats)
    n = 300_000
    texts = [_text(rng, BYTES, n, pats) for _ in range(3)]
    wants = [oracle.bucketed(t, pats, threads=8) for t in texts]
    cap = max(w.n for w in wants)
    dev = torch.from_numpy(texts[0]).cuda()
    out = torch.empty(cap * 16, dtype=torch.uint8, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = pf.Workspace()
    ws.reserve(n, 1, cap)
    side = torch.cuda.Stream()

    def scan(stream):
        if noalloc:
            pf.pfac_scan_noalloc(trie, dev, n, out, cap, cnt, None, stream)
        else:
            pf.pfac_scan(trie, ws, dev, n, out, cap, cnt, None, stream)

    if noalloc:  # (the first call on a device looks its array up)
        scan(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="thread_local"):
        scan(side)
    for i in (1, 2, 0, 1):
        # an eager scan of the same workspace first: nothing was cleared by the capture
        if not noalloc:
            got, _ = gpu_scan(trie, texts[i][:90_000 + i], ws=ws, counts=False)
            assert_same(got, oracle.bucketed(texts[i][:90_000 + i], pats, threads=8))
        dev.copy_(torch.from_numpy(texts[i]))
        out.fill_(0xAB)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(cnt.item()) == wants[i].n
        assert_same(pf.matches_to_numpy(out, wants[i].n), wants[i])
