"""Persistent plain steps whose planes are not a multiple of the 8 XCDs: with
the idle rows that put a chunk's consumer and producer on one XCD (the
library's grid), and without them (the fallback library), where every pair
hands its slots over between XCDs. Where the waves ran is read back."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from sifar_harness import StepRun, pairs_across, to_host

pytestmark = pytest.mark.gpu


# 45, 2 and 10 chunks; one token of 9; and 4095 chunks, where the padded grid
# holds more workgroups than the GPU has places (the idle rows end at once)
@pytest.mark.parametrize("N,T,H,L", [(8, 5, 4608, 12), (8, 1, 1024, 12), (3, 1, 5120, 11),
                                     (1, 1, 4608, 4), (2, 455, 4608, 4)])
def test_persistent_steps_on_odd_planes(grid, N, T, H, L):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    w = synth.Workload(81, f"planes-{N}-{T}-{H}", N, (T,), H, L, 1, "normal")
    run = StepRun(w, T, persistent=1)
    try:
        for rep in range(6 if T < 100 else 2):
            print(f"{grid} N={N} T={T} H={H} rep {rep}", flush=True)
            epochs = run.step(T)
            got = to_host(run.out_d)
            exp = oracle.reduce_chain(run.pool, epochs, T)
            for i in range(L):
                assert np.array_equal(got[i, :T], exp[i]), f"rep={rep} node={i}"
            across = pairs_across(run, T)
            print(f"pairs on two XCDs: {across:.3f}", flush=True)
            assert across == (0.0 if grid == "padded" else 1.0)
        run.s.check()
    finally:
        run.s.close()
