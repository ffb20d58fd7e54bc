"""Residual-add + RMSNorm at every kind of exchange width: one chunk per token
(no exchange), two, an odd number, one lane row of 16, one more, 33 and 64 (the
most), with rows that end inside a lane group and one of 8 elements; persistent
steps, per-epoch steps in one launch, and as launches of several workgroup
widths, four chained nodes, two steps. Residual bit-exact, y within 1 bf16 step
of the float64 oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from sifar_harness import StepRun, to_host, ulp_distance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("persistent,G,fuse", [(1, 1, 1), (0, 1, 1), (0, 1, 0), (0, 2, 0),
                                               (0, 16, 0)])
@pytest.mark.parametrize("H", [8, 512, 520, 3 * 512, 16 * 512, 16 * 512 + 8, 33 * 512 - 8, 64 * 512])
def test_epilogue_exchange_widths(H, persistent, G, fuse):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, T, L = 3, 5, 4
    w = synth.Workload(86, f"epilogue-width-{H}", N, (T,), H, L, 2, "act", epilogue=True)
    run = StepRun(w, T, persistent=persistent, waves_per_group=G, fuse_peers=fuse,
                  pool=synth.payload_pool(w.wid, N, T, H, 5, w.dist))
    res = run.res0.copy()
    for step in range(2):
        print(f"epilogue H={H} persistent={persistent} G={G} fuse={fuse} step {step}", flush=True)
        epochs = run.step(T)
        y_got = to_host(run.y_d)
        _, r_list, y_list = oracle.reduce_chain(run.pool, epochs, T,
                                                epilogue=(res, run.weight, w.rms_eps))
        assert np.array_equal(to_host(run.res_d), r_list[-1])
        for i in range(L):
            assert ulp_distance(y_got[i], y_list[i]).max() <= 1, f"step {step} node {i}"
        res = r_list[-1]
    run.s.check()
    run.s.close()
