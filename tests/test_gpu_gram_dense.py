"""Units of many matches in the gram kernel, against the oracle record by
record: past the short LDS lists that go with a large bitmap (every wave's
lists at another LDS address), in units of one chunk up to a dozen, so that
matches lie on both sides of unit position 8,192, below and above what the
unit's list in global memory holds."""

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


# 200 patterns: a bitmap of 4 KiB and long lists (64 or 160 matches a unit in
# LDS); 20,000: 128 KiB and short lists.  Units have 1, 1, 3 and 12 chunks, and
# their lists in global memory 32 entries a chunk: a match every 40 bytes fits
# them, one every 13 does not.
@pytest.mark.parametrize("n", [200_003, 2 * MiB, 9 * MiB + 5, 48 * MiB + 77])
@pytest.mark.parametrize("k,lo", [(200, 8), (20_000, 8), (20_000, 5)])
@pytest.mark.parametrize("step", [40, 13])
def test_dense_units(k, lo, n, step):
    rng = np.random.default_rng(k + lo + step)
    pats = [rng.integers(0, 256, int(rng.integers(lo, 14)), dtype=np.uint8).tobytes() for _ in range(k)]
    text = rng.integers(0, 256, n, dtype=np.uint8)
    for at0 in (0, n // 2 + 1, n - 70_000):
        for q in range(min(3000, 60_000 // step)):
            p = np.frombuffer(pats[(q * 7) % k], dtype=np.uint8)
            at = at0 + q * step
            text[at:at + p.size] = p
    want = oracle.bucketed(text, pats, threads=8)
    say(f"gram dense units k={k} lo={lo} n={n} step={step}: {want.n} matches")
    got, counts = gpu_scan(pf.Trie(pats), text, pad_front=5)
    assert_same(got, want)
    assert np.array_equal(counts, oracle.counts(n, want))
