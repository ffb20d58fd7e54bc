"""The allocation-free all-reduce in one launch: edges of its range (8 elements,
the widest row, 64 tokens, ragged rows, padded rank strides, every rank count's
ends), and replays of a captured call on changing inputs with eager calls
between them, all bit-exact against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2607_08973_amd as S
import synth
from sifar_harness import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"


@pytest.mark.parametrize("N,T,H,pad", [(1, 1, 8, 0), (8, 1, 512, 8), (2, 1, 520, 0), (8, 4, 65536, 0),
                                       (7, 64, 4088, 16), (3, 64, 4096, 0), (8, 33, 1000, 4096)])
def test_noalloc_edges(N, T, H, pad):
    x = synth.bf16(synth.rng(91, N, T, H), (3, N, T, H), "act")
    for rep in range(3):
        print(f"noalloc N={N} T={T} H={H} pad={pad} rep {rep}", flush=True)
        src = torch.zeros((N, T * H + pad), dtype=torch.int16, device=DEV)
        src[:, :T * H] = to_dev(x[rep]).reshape(N, T * H)
        out = torch.full((T, H), -1, dtype=torch.int16, device=DEV)
        S.sifar_allreduce_noalloc(src, T * H + pad, N, T, H, out)
        assert np.array_equal(to_host(out), oracle.reduce(x[rep]))


def test_noalloc_captured_call_replays():
    N, T, H = 8, 5, 4104
    x = synth.bf16(synth.rng(92), (6, N, T, H), "act")
    src, out = to_dev(x[0]), torch.zeros((T, H), dtype=torch.int16, device=DEV)
    other = torch.zeros((T, H), dtype=torch.int16, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        S.sifar_allreduce_noalloc(src, T * H, N, T, H, out)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.sifar_allreduce_noalloc(src, T * H, N, T, H, out)
    for i in range(6):
        print(f"noalloc replay {i}", flush=True)
        src.copy_(to_dev(x[i]))
        graph.replay()
        y = to_dev(x[5 - i])
        S.sifar_allreduce_noalloc(y, T * H, N, T, H, other)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(out), oracle.reduce(x[i])), i
        assert np.array_equal(to_host(other), oracle.reduce(x[5 - i])), i


# in place over one rank's partial; the output some rows, one vector or one
# whole chunk before or after the sources; and across two ranks' partials
@pytest.mark.parametrize("N,T,H", [(8, 64, 4096), (3, 7, 1000), (2, 4, 65536)])
@pytest.mark.parametrize("where", ["rank0", "last", "vector", "chunk", "before", "rows", "across"])
def test_noalloc_output_over_the_sources(N, T, H, where):
    K = T * H
    at = {"rank0": 0, "last": (N - 1) * K, "vector": 8, "chunk": 512, "before": -8, "rows": H,
          "across": K // 2 // 8 * 8}[where]
    x = synth.bf16(synth.rng(97, N, T, H), (2, N, T, H), "act")
    for rep in range(2):
        print(f"noalloc N={N} T={T} H={H} out at {where} rep {rep}", flush=True)
        buf = torch.zeros(8 + N * K + K, dtype=torch.int16, device=DEV)
        buf[8:8 + N * K] = to_dev(x[rep]).reshape(-1)
        out = buf[8 + at:8 + at + K]
        S.sifar_allreduce_noalloc(buf[8:], K, N, T, H, out)
        assert np.array_equal(to_host(out).reshape(T, H), oracle.reduce(x[rep]))
