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


TESTS = [lists_aligned]


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
