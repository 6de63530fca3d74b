"""The host side of scans without a GPU: what the library allocates, clears,
launches and waits for, seen through HIP entry points over host memory
(native/host_hip.cpp).  Each test runs in a process of its own, since those
entry points have to be in place before libpfac.so is loaded."""

import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
TEXT, OUT, COUNT, OFFSETS = 0x10000, 0x20000000000, 0x30000, 0x40000  # device addresses, never read
KiB, MiB = 1 << 10, 1 << 20


@pytest.fixture(scope="module")
def host_hip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host_hip") / "host_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "native", "host_hip.cpp"), "-o", so], check=True)
    return so


def _child(host_hip, name):
    run = subprocess.run([sys.executable, os.path.abspath(__file__), host_hip, name], capture_output=True, text=True,
                         timeout=300, cwd=ROOT)
    assert run.returncode == 0, (run.stdout + run.stderr)[-4000:]


# ---------------------------------------------------------------- the children


def _lines():
    out = hip.host_hip_text().decode().splitlines()
    hip.host_hip_clear()
    return out


def _launches(lines=None):
    """(kernel, grid, block, dynamic LDS) of each launch."""
    found = []
    for ln in _lines() if lines is None else lines:
        m = re.match(r"launch grid (\d+) block (\d+) lds (\d+) stream (\d+) _ZN4pfac\d+([a-z_0-9]+?)(I|E)", ln)
        if m:
            found.append((m[5], int(m[1]), int(m[2]), int(m[3])))
    return found


def _bytes_set(k, lo=8, hi=40, seed=1):
    rng = np.random.default_rng(seed)
    return [rng.integers(0, 256, int(rng.integers(lo, hi + 1)), dtype=np.uint8).tobytes() for _ in range(k)]


def lists_aligned():
    """A wave reads sixteen bytes at a time from the start of its LDS lists:
    they begin at multiples of sixteen for every wave, behind a bitmap of any
    size and without one."""
    for k in (200, 2000, 20_000):
        trie = pf.Trie(_bytes_set(k))
        for n in (64 * KiB, 2 * MiB, 16 * MiB):
            _lines()
            pf.pfac_scan(trie, pf.Workspace(), TEXT, n, OUT, 100, COUNT)
            (_, _, block, lds), = [x for x in _launches() if x[0] == "scan_grams"]
            waves = block // 64
            bits = 1 << 12
            while bits < min(24 * 4 * k, 1 << 20):
                bits *= 2
            table = bits // 8 if n > 2560 * KiB or bits // 8 <= 16 * KiB else 0
            assert (lds - 16 - table) % (16 * waves) == 0, (k, n, lds, waves)


def _kernels(lines=None):
    return [name for name, *_ in _launches(lines)]


def cursor_cleared():
    """The staging cursor of a new workspace is cleared by its first scan, on
    the scan's own stream (streams need not wait for the one that a clearing at
    creation would take), a captured scan leaves that to the next one too, and
    later scans have nothing to clear unless a launch failed."""
    trie = pf.Trie(_bytes_set(500))
    stream = 0x770

    def scan(ws):
        pf.pfac_scan(trie, ws, TEXT, 5000, OUT, 100, COUNT, stream=stream)

    ws = pf.Workspace()
    assert not [ln for ln in _lines() if ln.startswith("memset")]
    scan(ws)
    lines = _lines()
    assert _kernels(lines) == ["reset_kernel", "scan_grams", "finish_tiles"]
    assert all(f"stream {stream} " in ln for ln in lines if ln.startswith("launch"))
    scan(ws)
    assert _kernels() == ["scan_grams", "finish_tiles"]

    ws = pf.Workspace()
    ws.reserve(5000, 1, 100)
    _lines()
    hip.host_hip_capture(1)
    scan(ws)
    hip.host_hip_capture(0)
    assert _kernels() == ["reset_kernel", "scan_grams", "finish_tiles"]
    scan(ws)
    assert _kernels() == ["reset_kernel", "scan_grams", "finish_tiles"]
    scan(ws)
    assert _kernels() == ["scan_grams", "finish_tiles"]

    def noalloc():
        pf.pfac_scan_noalloc(trie, TEXT, 5000, OUT, 100, COUNT, stream=stream)

    for call in (lambda: scan(ws), noalloc):
        call()
        hip.host_hip_refuse(b"finish_tiles")
        _lines()
        with pytest.raises(pf.PfacError) as e:
            call()
        assert e.value.code == pf.PFAC_EDEVICE
        # at once, for replays of scans captured before, and again with the next
        assert _kernels() == ["scan_grams", "reset_kernel"]
        hip.host_hip_refuse(b"")
        call()
        assert _kernels() == ["reset_kernel", "scan_grams", "finish_tiles"]
        call()
        assert _kernels() == ["scan_grams", "finish_tiles"]


def graph_cursor_cleared():
    """A graph's own workspace is cleared, and the clearing waited for, before
    its scan is captured: replays have nothing to clear."""
    trie = pf.Trie(_bytes_set(500))
    _lines()
    pf.Graph(trie, None, TEXT, OFFSETS, 10, 5000, OUT, 100, COUNT)
    lines = [ln for ln in _lines() if ln.startswith(("launch", "capture", "sync", "memset"))]
    at = lines.index("capture begins")
    assert _kernels(lines[:at]) == ["reset_kernel"] and lines[at - 1].startswith("sync stream ")
    assert lines[at - 1].split()[2] == re.search(r"stream (\d+)", lines[at - 2])[1]
    assert _kernels(lines[at:]) == ["plan_kernel", "scan_grams", "finish_tiles"]


def reserved_scans_allocate_nothing():
    """After pfac_workspace_reserve no scan allocates, device memory or pinned
    memory; a synchronous scan waits once and copies nothing.  A call that is
    refused touches nothing either, and graphs (which have no synchronous scans)
    take no pinned memory."""
    for pats in (_bytes_set(500), [b"ab", b"abc", b"xyz"]):
        trie = pf.Trie(pats)
        ws = pf.Workspace()
        ws.reserve(20 * MiB, 10, 1000)
        _lines()
        for n in (1460, 64 * KiB, 20 * MiB):
            for _ in range(2):
                pf.pfac_scan_sync(trie, ws, TEXT, n, OUT, 1000)
                lines = _lines()
                assert not [ln for ln in lines if "malloc" in ln or ln.startswith("copy")], (n, lines)
                assert [ln for ln in lines if ln.startswith("sync")] == ["sync stream 0"]
            pf.pfac_scan(trie, ws, TEXT, n, OUT, 1000, COUNT)
            pf.pfac_scan_batch(trie, ws, TEXT, OFFSETS, 3, n, OUT, 1000, COUNT)
            assert not [ln for ln in _lines() if "malloc" in ln]
    host_only = pf.Trie(_bytes_set(500), host_only=True)
    for t in (host_only, trie):
        fresh = pf.Workspace()
        _lines()
        with pytest.raises(pf.PfacError) as e:
            pf.pfac_scan_sync(t, fresh, None, 100, OUT, 1000)
        assert e.value.code == (pf.PFAC_EINVAL if t is trie else pf.PFAC_ENODEV)
        assert not _lines()
    pf.Graph(trie, None, TEXT, OFFSETS, 10, 5000, OUT, 100, COUNT)
    assert not [ln for ln in _lines() if ln.startswith("host malloc")]


def _areas(lines):
    return [int(ln.split()[1]) for ln in lines if ln.startswith("malloc ")]


def first_scan_allocates_what_it_reads():
    """The first scan of a workspace allocates no more areas than the tile
    kernel does, whose launches the gram kernel took over: counts, offsets and
    first texts per unit, the staging area, the inline slots and the list area
    (in place of the chunks' boundaries and the block sums)."""
    trie = pf.Trie(_bytes_set(500))
    for n in (1460, 5_000_011):
        calls = [lambda ws: pf.pfac_scan(trie, ws, TEXT, n, OUT, 100, COUNT),
                 lambda ws: pf.pfac_scan_batch(trie, ws, TEXT, OFFSETS, 3, n, OUT, 100, COUNT),
                 lambda ws: pf.pfac_scan_batch_plain(trie, ws, TEXT, np.array([0, n], dtype=np.uint64), 1, OUT, 100,
                                                     COUNT)]
        for call in calls:
            ws = pf.Workspace()
            _lines()
            call(ws)
            lines = _lines()
            assert "scan_grams" in _kernels(lines)
            assert len(_areas(lines)) == 6, lines
        _lines()
        pf.Graph(trie, None, TEXT, OFFSETS, 3, n, OUT, 100, COUNT)
        assert len(_areas(_lines())) == 1 + 6  # and the cursor's


def list_area_refused():
    """Where the device cannot hold the gram kernel's list area (512 bytes a
    KiB), the kernels that ran these scans without one still do; the workspace
    asks again only when it is reserved anew, so captured scans after a first
    one find it ready."""
    n = 5_000_011
    words = [bytes(np.random.default_rng(i).choice(np.arange(97, 107), 9).astype(np.uint8)) for i in range(300)]
    offsets = np.array([0, n // 3, n], dtype=np.uint64)
    for pats, kernel in ((_bytes_set(500), "scan_tiles"), (words, "scan_waves")):
        trie = pf.Trie(pats)
        for call in (lambda: pf.pfac_scan(trie, ws, TEXT, n, OUT, 100, COUNT),
                     lambda: pf.pfac_scan_sync(trie, ws, TEXT, n, OUT, 100),
                     lambda: pf.pfac_scan_batch(trie, ws, TEXT, OFFSETS, 2, n, OUT, 100, COUNT),
                     lambda: pf.pfac_scan_batch_plain(trie, ws, TEXT, offsets, 2, OUT, 100, COUNT),
                     lambda: pf.Graph(trie, None, TEXT, OFFSETS, 2, n, OUT, 100, COUNT)):
            ws = pf.Workspace()
            hip.host_hip_limit(1 * MiB)
            _lines()
            call()
            lines = _lines()
            assert kernel in _kernels(lines) and "scan_grams" not in _kernels(lines), lines
            hip.host_hip_limit(1 << 40)
        call = lambda: pf.pfac_scan(trie, ws, TEXT, n, OUT, 100, COUNT)  # noqa: E731
        ws = pf.Workspace()
        hip.host_hip_limit(1 * MiB)
        call()
        _lines()
        call()
        lines = _lines()
        assert not [ln for ln in lines if "malloc" in ln or ln.startswith("sync")]
        assert kernel in _kernels(lines)
        with pytest.raises(pf.PfacError) as e:
            ws.reserve(n, 1, 100)
        assert e.value.code == pf.PFAC_ENOMEM
        hip.host_hip_limit(1 << 40)
        ws.reserve(n, 1, 100)
        _lines()
        call()
        assert "scan_grams" in _kernels()
        # the split kernels always needed theirs
        ws = pf.Workspace()
        hip.host_hip_limit(6 * MiB)
        if kernel == "scan_tiles":
            with pytest.raises(pf.PfacError) as e:
                pf.pfac_scan(trie, ws, TEXT, 16 * MiB, OUT, 100, COUNT)
            assert e.value.code == pf.PFAC_ENOMEM
        hip.host_hip_limit(1 << 40)


def explicit_kernels_run():
    """Kernels 0, 1 and 2 mean what they say, also where a call sets the very
    values that the build chose; kernel 3, and a trie whose tuning was never
    set, leave the choice to the library."""
    rng = np.random.default_rng(3)
    words = [bytes(rng.choice(np.arange(97, 107), 9).astype(np.uint8)) for _ in range(300)]
    main = {0: "scan_tiles", 1: "scan_waves", 2: "scan_waves", 3: "scan_grams"}

    def ran(trie, n=9 * MiB):
        _lines()
        pf.pfac_scan(trie, pf.Workspace(), TEXT, n, OUT, 100, COUNT)
        lines = _lines()
        name, = [k for k in _kernels(lines) if k in main.values()]
        return name, "walk_units" in _kernels(lines)

    for pats, chosen in ((words, 1), (_bytes_set(500), 3), ([b"ACGTACGTAC" + bytes([c]) for c in b"ACGT"], 1)):
        trie = pf.Trie(pats)
        built = trie.tuning()
        assert built["kernel"] == chosen
        assert ran(trie) == ("scan_grams", False)
        for kernel in (chosen, 0, 1, 2, 3, 1):
            trie.set_tuning(kernel=kernel)
            assert trie.tuning() == dict(built, kernel=kernel)
            assert ran(trie) == (main[kernel], kernel == 2)
        # other fields of a tuning are a choice as well
        trie = pf.Trie(pats)
        trie.set_tuning(waves_per_wg=8)
        assert ran(trie)[0] == main[chosen]

    # the autotuner times the library's choice and each kernel under its own name
    trie = pf.Trie(words)
    best = pf.pfac_autotune(trie, pf.Workspace(), TEXT, 9 * MiB)
    assert best["kernel"] == 3 and best == trie.tuning()  # all took as long here: the first one stays
    names = [k for k in _kernels() if k in main.values()]
    first = next(i for i, k in enumerate(names) if k != "scan_grams")
    assert 0 < first < 20 and "scan_grams" not in names[first:] and {"scan_tiles", "scan_waves"} <= set(names)
    assert ran(trie)[0] == "scan_grams"


def small_alphabets():
    """The gram kernel runs the sets over small alphabets that it scans faster
    than the fused kernel, of random texts: few patterns, or many matches."""
    for symbols, k, lo, hi, kernel in ((6, 30, 8, 16, "scan_grams"), (6, 300, 8, 16, "scan_waves"),
                                       (8, 1000, 6, 10, "scan_waves"), (12, 300, 8, 16, "scan_grams"),
                                       (12, 3000, 8, 16, "scan_waves"), (16, 10_000, 8, 16, "scan_grams"),
                                       (20, 30_000, 8, 16, "scan_grams"), (26, 30_000, 6, 10, "scan_grams"),
                                       (6, 100, 4, 8, "scan_grams"), (40, 30_000, 8, 16, "scan_grams")):
        rng = np.random.default_rng(symbols)
        a = np.arange(48, 48 + symbols)
        trie = pf.Trie([bytes(rng.choice(a, int(m)).astype(np.uint8)) for m in rng.integers(lo, hi + 1, k)])
        _lines()
        pf.pfac_scan(trie, pf.Workspace(), TEXT, 32 * MiB, OUT, 100, COUNT)
        assert kernel in _kernels(), (symbols, k, lo)


def launch_gram_tells():
    """pfac_trie_launch_gram says of every launch whether the gram kernel runs
    it, and how; the bench names the main kernel by it."""
    import bench

    rng = np.random.default_rng(5)
    dna = np.frombuffer(b"ACGT", dtype=np.uint8)
    sets = [_bytes_set(300), _bytes_set(20_000), _bytes_set(300, lo=3), _bytes_set(9000, lo=4), _bytes_set(6000, lo=5),
            [bytes(rng.choice(dna, 9)) for _ in range(100)], [bytes(rng.choice(dna, 20)) for _ in range(40_000)],
            [bytes(rng.choice(dna, int(m))) for m in rng.integers(20, 33, 200_000)],  # beyond the filter
            [bytes(rng.choice(np.arange(97, 107), 9).astype(np.uint8)) for _ in range(300)]]
    seen = set()
    for pats in sets:
        trie = pf.Trie(pats)
        for tuning in ({}, dict(kernel=1), dict(kernel=3), dict(kernel=3, trunc_depth=8), dict(kernel=3, dag=1, trunc_depth=0)):
            if tuning:
                if len(pats) > 50_000:
                    continue
                trie.set_tuning(**tuning)
            for n in (1460, 2 * MiB, 2 * MiB + MiB // 2 + KiB, 40 * MiB):
                told = trie.launch_gram(n)
                _lines()
                pf.pfac_scan(trie, pf.Workspace(), TEXT, n, OUT, 100, COUNT)
                (name, grid, block, lds), = [x for x in _launches() if x[0] in ("scan_grams", "scan_waves", "scan_tiles")]
                assert (told["step"] != 0) == (name == "scan_grams"), (len(pats), tuning, n)
                st = dict(launch_gram=told["step"], launch_kernel=trie.launch_kernel(n)[0])
                assert bench.kernel_of(st)[0] == name
                if told["step"]:
                    assert block == 64 * told["waves_per_wg"] and lds == told["lds_bytes"]
                    assert lds > told["bitmap_bytes"] or not told["bitmap_in_lds"]
                    units = -(-n // (KiB * told["chunks_per_unit"]))
                    assert grid == min(-(-units // told["waves_per_wg"]), 256 if told["bitmap_in_lds"] else 1 << 30)
                    seen.add((told["step"], bool(told["symbols"]), told["runs"], told["bitmap_in_lds"]))
    assert {(s, False, 0, b) for s in (1, 2, 4) for b in (0, 1)} <= seen and {(1, True, 1, 0), (1, True, 1, 1)} <= seen
    assert pf.load().pfac_trie_launch_gram(None, 1, None) == pf.PFAC_EINVAL
    assert pf.load().pfac_trie_launch_gram(trie.handle, 1, None) == pf.PFAC_EINVAL


def noalloc_routes():
    """pfac_scan_noalloc takes the gram kernel while its list area fits in the
    64 MiB beside the records, then the kernels that need less; what fits
    neither is refused before anything is launched."""
    trie = pf.Trie(_bytes_set(3000))
    n = 7 * MiB + 5
    for cap, kernel in ((1000, "scan_grams"), ((58 * MiB) // 16, "scan_grams"), ((62 * MiB) // 16, "scan_tiles")):
        _lines()
        pf.pfac_scan_noalloc(trie, TEXT, n, OUT, cap, COUNT)
        lines = _lines()
        assert kernel in _kernels(lines) and not _areas(lines)
    with pytest.raises(pf.PfacError) as e:
        pf.pfac_scan_noalloc(trie, TEXT, n, OUT, 4 * MiB, COUNT)
    assert e.value.code == pf.PFAC_EINVAL and not _lines()


TESTS = [noalloc_routes, launch_gram_tells, small_alphabets, explicit_kernels_run, list_area_refused, first_scan_allocates_what_it_reads, lists_aligned, cursor_cleared, graph_cursor_cleared, reserved_scans_allocate_nothing]


@pytest.mark.parametrize("name", [t.__name__ for t in TESTS])
def test_host(host_hip, name):
    _child(host_hip, name)


if __name__ == "__main__":
    hip = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
    hip.host_hip_text.restype = ctypes.c_char_p
    hip.host_hip_limit.argtypes = [ctypes.c_size_t]
    hip.host_hip_room.argtypes = [ctypes.c_void_p]
    hip.host_hip_room.restype = ctypes.c_size_t
    hip.host_hip_refuse.argtypes = [ctypes.c_char_p]
    sys.path.insert(0, ROOT)
    import paper_1702_03657_amd as pf

    globals()[sys.argv[2]]()
