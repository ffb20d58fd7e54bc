"""Calls whose answer must not depend on which kernels run a per-epoch step:
the one-launch step against separate producer and reduction launches
(fuse_peers = 0) and the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2607_08973_amd as S
import synth
from sifar_harness import StepRun, inject_table, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"


# forced retries that use the budget up, and a withheld rank beside a late one;
# H of one chunk and of nine
@pytest.mark.parametrize("mode", ["spec", "ordered"])
@pytest.mark.parametrize("N,T,H,forced,withheld", [(4, 2, 512, 0, 0b0100), (8, 3, 4608, 0, 0b1000),
                                                   (3, 2, 1032, 9, 0)])
def test_output_of_an_exhausted_budget_is_the_last_load(N, T, H, forced, withheld, mode):
    """Epoch 3: rank 0 is late and catches up after the first validation, but
    the chunk's budget of 3 runs out (a withheld stamp, or more forced retries
    than attempts). What is stored is the sum of the last load, in which rank 0
    has caught up -- every payload is in place, so it equals the oracle's."""
    L = 4
    w = synth.Workload(95, f"budget-{N}-{H}", N, (T,), H, L, 1, "normal")
    late, held = np.array([0, 0, 1, 0]), np.array([0, 0, withheld, 0])
    a = StepRun(w, T, validate=mode, max_attempts=3, forced_retries=forced)
    b = StepRun(w, T, validate=mode, max_attempts=3, forced_retries=forced, fuse_peers=0,
                pool=a.pool)
    outs = []
    for r in (a, b):
        print(f"exhausted budget N={N} H={H} forced={forced} {mode}", flush=True)
        r.s.set_injection(inject_table(late, withheld=held))
        r.step(T)
        assert r.s.status() == S.SIFAR_EDEVICE
        kind, _, _, attempts = r.s.error_info()
        assert (kind, attempts) == (S.SIFAR_DEV_RETRY_BUDGET, 3)
        outs.append(to_host(r.out_d))
        r.s.close()
    assert np.array_equal(outs[1][2], oracle.reduce(a.pool[2]))
    assert np.array_equal(outs[0], outs[1])


# a token of four, of 16, and of one chunk (four consumer waves)
@pytest.mark.parametrize("H,T,G", [(2048, 32, 4), (8192, 8, 16), (512, 3, 1)])
def test_whole_token_workgroups_need_no_spin_limit(H, T, G):
    """With waves per workgroup that hold a whole token, the epilogue's launches
    add a token's sum of squares without a wait between workgroups, so any
    spin_limit does; so it must in a one-launch step."""
    N, L, steps = 8, 8, 25
    w = synth.Workload(96, f"spin-{H}", N, (T,), H, L, 1, "act", epilogue=True)
    runs = [StepRun(w, T, waves_per_group=G, spin_limit=1, fuse_peers=f,
                    pool=synth.payload_pool(96, N, T, H, 5, "act")) for f in (1, 0)]
    for step in range(steps):
        if step % 5 == 0:
            print(f"whole-token workgroups H={H} T={T} G={G} step {step}", flush=True)
        for r in runs:
            r.step(T)
            r.s.check()
        assert np.array_equal(to_host(runs[0].res_d), to_host(runs[1].res_d)), step
    for r in runs:
        r.s.close()
