"""Calls without a stream run on the caller's current stream of the current
device, also inside a stream context and after it."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2607_08973_amd as S
import synth
from sifar_harness import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, T, H = 4, 3, 1000
    x = synth.bf16(synth.rng(93), (4, N, T, H), "act")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert S._stream(None) == torch.cuda.current_stream().cuda_stream
    with S.Sifar(nranks=N, hidden=H, max_tokens=T, reduces_per_step=1) as s:
        for i, st in enumerate((None, side, None, side)):
            src, out = torch.zeros((N, T, H), dtype=torch.int16, device=DEV), torch.zeros(
                (T, H), dtype=torch.int16, device=DEV)
            torch.cuda.synchronize()
            with torch.cuda.stream(st):
                assert S._stream(None) == torch.cuda.current_stream().cuda_stream
                # the copy is on the same stream: a call on another would read zeros
                src.copy_(to_dev(x[i]), non_blocking=True)
                s.produce(src, T)
                s.reduce(out, T)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(out), oracle.reduce(x[i])), i
        s.check()
