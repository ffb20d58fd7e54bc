"""Persistent plain steps whose planes are not a multiple of the 8 XCDs: with
the idle rows that put a chunk's consumer and producer on one XCD (the
library's grid), and without them (a copy of the library built for this test),
so that every pair hands its slots over between XCDs."""
from __future__ import annotations

import os

import numpy as np
import pytest
import torch

import oracle
import paper_2607_08973_amd as S
import synth
from sifar_harness import StepRun, to_host

pytestmark = pytest.mark.gpu

UNPADDED = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libsifar_unpadded.so")


@pytest.fixture(params=["padded", "unpadded"])
def library(request, monkeypatch):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    if request.param == "unpadded":
        monkeypatch.setattr(S, "_lib", None)
        S.load(UNPADDED)
    yield request.param


# 45, 2 and 10 chunks; one token of 9; and 4095 chunks, where the padded grid
# holds more workgroups than the GPU has places (the idle rows end at once)
@pytest.mark.parametrize("N,T,H,L", [(8, 5, 4608, 12), (8, 1, 1024, 12), (3, 1, 5120, 11),
                                     (1, 1, 4608, 4), (2, 455, 4608, 4)])
def test_persistent_steps_on_odd_planes(library, N, T, H, L):
    w = synth.Workload(81, f"planes-{N}-{T}-{H}", N, (T,), H, L, 1, "normal")
    run = StepRun(w, T, persistent=1)
    try:
        for rep in range(6 if T < 100 else 2):
            print(f"{library} N={N} T={T} H={H} rep {rep}", flush=True)
            epochs = run.step(T)
            got = to_host(run.out_d)
            exp = oracle.reduce_chain(run.pool, epochs, T)
            for i in range(L):
                assert np.array_equal(got[i, :T], exp[i]), f"rep={rep} node={i}"
        run.s.check()
    finally:
        run.s.close()
