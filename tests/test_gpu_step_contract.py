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
from sifar_harness import DEV, StepRun, inject_table, to_dev, to_host

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


def _flat_step(N, P, T, H, L, ring_at, fuse, seed=98):
    """A step whose pool and ring lie in one flat buffer, the ring `ring_at`
    elements from its start; returns the flat buffer's contents before the step
    and after each of two steps."""
    K = T * H
    pool = synth.payload_pool(seed, N, T, H, P, "act")
    flat = torch.zeros(max(P * N * K, ring_at + L * K), dtype=torch.int16, device=DEV)
    flat[:P * N * K] = to_dev(pool).reshape(-1)
    states = [to_host(flat)]
    with S.Sifar(nranks=N, hidden=H, max_tokens=T, reduces_per_step=L, fuse_peers=fuse) as s:
        S.sifar_bind_step(s.h, flat, P, N * K, K, out_ring=flat[ring_at:])
        assert s.step_plan(T)[0] == L + 2   # not in one launch
        for _ in range(2):
            s.step(T)
            s.check()
            states.append(to_host(flat))
    return states


# one rank: all-reduce i's output becomes (part of) the partial of a later
# epoch, at the same chunks and shifted by a vector; two ranks: outputs over
# partials that were read before
@pytest.mark.parametrize("N,P,L,at,shift", [(1, 9, 5, 2, 0), (1, 10, 6, 2, 8), (1, 12, 6, 4, 512),
                                            (2, 12, 6, 0, 0), (2, 12, 6, 0, 8)])
@pytest.mark.parametrize("T,H", [(64, 4096), (3, 1000)])
def test_outputs_over_the_source_pool(N, P, L, at, shift, T, H):
    """The step runs one all-reduce after the other over whatever the buffers
    hold: what an output overwrote is what a later epoch reads."""
    K = T * H
    ring_at = at * N * K + shift
    print(f"outputs over the pool N={N} P={P} L={L} ring at {ring_at} T={T} H={H}", flush=True)
    states = _flat_step(N, P, T, H, L, ring_at, 1)
    mem = states[0].copy()
    for step in range(2):
        for i in range(L):
            e = (step * (L + L % 2) + i) % P     # an odd chain skips an epoch
            x = mem[e * N * K:(e + 1) * N * K].reshape(N, T, H)
            mem[ring_at + i * K:ring_at + (i + 1) * K] = oracle.reduce(x).reshape(-1)
        assert np.array_equal(states[1 + step], mem), f"step {step}"


@pytest.mark.parametrize("alias", ["residual", "weight"])
def test_epilogue_outputs_over_its_own_inputs(alias):
    """y of all-reduce 1 overwrites the residual, or the weight, that the next
    ones read: word for word what separate launches do."""
    N, T, H, L = 4, 1, 4096, 5
    pool = to_dev(synth.payload_pool(99, N, T, H, 7, "act"))
    out = []
    for fuse in (1, 0):
        y = torch.zeros((L, T, H), dtype=torch.int16, device=DEV)
        res, wgt = to_dev(synth.residual_init(99, T, H)), to_dev(synth.rms_weight(99, H))
        if alias == "residual":
            y[1].copy_(res)
            res = y[1]
        else:
            y[1, 0].copy_(wgt)
            wgt = y[1, 0]
        with S.Sifar(nranks=N, hidden=H, max_tokens=T, reduces_per_step=L, epilogue=1,
                     fuse_peers=fuse) as s:
            s.bind_step(pool, residual=res, weight=wgt, y_ring=y)
            for _ in range(2):
                print(f"epilogue over its {alias} fuse={fuse}", flush=True)
                s.step(T)
                s.check()
        out.append((to_host(y), to_host(res)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("capture_mode", ["global", "thread_local", "relaxed"])
@pytest.mark.parametrize("epilogue", [False, True])
@pytest.mark.parametrize("fuse", [1, 0])
def test_step_on_a_capturing_stream_is_not_recorded(fuse, epilogue, capture_mode):
    """On a capturing stream a per-epoch step runs at once, whichever kernels
    would otherwise run it, and the host's epochs stay the device's: replays of
    the (empty) capture change nothing and the next steps go on."""
    w = synth.Workload(100, "capture", 4, (3,), 1000, 4, 1, "act", epilogue=epilogue)
    run = StepRun(w, 3, fuse_peers=fuse, pool=synth.payload_pool(100, 4, 3, 1000, 23, "act"))
    res = run.res0.copy() if epilogue else None

    def check(epochs, what):
        nonlocal res
        torch.cuda.synchronize()
        run.s.check()
        assert run.s.epochs() == (epochs[-1] + 1, epochs[-1] + 1), what
        if epilogue:
            _, r, y = oracle.reduce_chain(run.pool, epochs, 3, epilogue=(res, run.weight, w.rms_eps))
            res = r[-1]
            assert np.array_equal(to_host(run.res_d), res), what
        else:
            exp = oracle.reduce_chain(run.pool, epochs, 3)
            assert np.array_equal(to_host(run.out_d), np.stack(exp)), what

    check(run.step(3), "first")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        graph.capture_begin(capture_error_mode=capture_mode)
        try:
            epochs = run.step(3)
        finally:
            graph.capture_end()
    check(epochs, "captured")
    for k in range(2):
        print(f"after a capture fuse={fuse} epilogue={epilogue} step {k}", flush=True)
        graph.replay()
        check(run.step(3), f"after replay {k}")
    run.s.close()
