"""The rules on overlapping buffers (csrc/spans.h) that keep a call off the
one-launch kernels, against byte maps of random small layouts. The header is
compiled for the host; no GPU is used."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

from paper_2607_08973_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_overlap_rules_match_byte_maps(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = tmp_path / "spans_check"
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", B.CSRC,
                    os.path.join(HERE, "spans_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr
