"""The tables of the gram filter as the builder makes them (CPU only, under
AddressSanitizer and UndefinedBehaviorSanitizer): every gram of every pattern
passes the bitmap, has its slot and a record that leads back to the pattern."""

import os
import shutil

import pytest

from tests.test_sanitizers import NATIVE, ROOT, SAN, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_gram_tables(tmp_path):
    out = _run(["g++", "-std=c++17", *SAN, os.path.join(NATIVE, "sanitize_grams.cpp"),
                os.path.join(ROOT, "paper_1702_03657_amd", "csrc", "trie_build.cpp")],
               tmp_path, "sanitize_grams")
    assert "ok" in out
