"""Per-epoch steps in one launch (dual buffers, peers one epoch ahead)
against the same steps as separate producer and reduction launches
(fuse_peers = 0) and the oracle: outputs, decision log and raw stamps must be
the same words, whatever the shape, validation mode, chain length, injected
late ranks, forced retries or waves per workgroup of the launches."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2607_08973_amd as S
import synth
from sifar_harness import StepRun, inject_table, to_host, ulp_distance

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _same_words(a, b, T, epochs):
    segs = a.s.log_geometry()[1]
    rows = [(g - 1) % a.L for g in epochs]
    la, lb = a.s.read_log()[rows, :T * segs], b.s.read_log()[rows, :T * segs]
    assert np.array_equal(la, lb), "decision logs"
    w = a.T_max * segs
    sa = a.s.read_stamp_log().reshape(a.L, w, 2, a.N)[rows, :T * segs]
    sb = b.s.read_stamp_log().reshape(b.L, w, 2, b.N)[rows, :T * segs]
    assert np.array_equal(sa, sb), "stamp logs"


# the smallest row, a row of one full and one 8-element chunk, ragged rows,
# many chunks; both sides of 256 chunks (four consumer waves per chunk, or one);
# chain lengths of 1, 2 and odd; every rank count's ends
@pytest.mark.parametrize("mode", ["spec", "ordered", "none"])
@pytest.mark.parametrize("N,T,H,L,G", [(4, 32, 4096, 3, 1), (4, 257, 504, 3, 1), (6, 37, 3592, 3, 2),
                                       (1, 1, 8, 1, 1), (8, 3, 520, 2, 2), (5, 7, 3896, 5, 16),
                                       (2, 9, 4608, 7, 4), (8, 64, 4096, 4, 1),
                                       (3, 130, 8192, 3, 8)])
def test_one_launch_equals_separate_launches(N, T, H, L, G, mode):
    w = synth.Workload(82, f"one-launch-{N}-{T}-{H}", N, (T,), H, L, 1, "act")
    a = StepRun(w, T, validate=mode, fuse_peers=1)
    b = StepRun(w, T, validate=mode, fuse_peers=0, waves_per_group=G, pool=a.pool)
    for tokens in (T, max(1, T // 2), T):
        print(f"one launch N={N} T={tokens} H={H} L={L} {mode}", flush=True)
        ea, eb = a.step(tokens), b.step(tokens)
        assert ea == eb
        got = to_host(a.out_d)
        exp = oracle.reduce_chain(a.pool, ea, tokens)
        for i in range(L):
            assert np.array_equal(got[i, :tokens], exp[i]), f"tokens={tokens} node={i}"
        _same_words(a, b, tokens, ea)
    for r in (a, b):
        r.s.check()
        r.s.close()


@pytest.mark.parametrize("mode", ["spec", "ordered"])
@pytest.mark.parametrize("N,T,H,forced", [(8, 2, 4096, 0), (3, 3, 1000, 2), (8, 1, 520, 1)])
def test_late_ranks_catch_up_the_same(N, T, H, forced, mode):
    L = 12
    w = synth.Workload(83, f"one-launch-late-{N}-{H}", N, (T,), H, L, 1, "act")
    late = synth.delay_table(83, N, 2 * L + 1, 0.3)
    a = StepRun(w, T, validate=mode, forced_retries=forced, fuse_peers=1)
    b = StepRun(w, T, validate=mode, forced_retries=forced, fuse_peers=0, pool=a.pool)
    for r in (a, b):
        r.s.set_injection(inject_table(late))
    for step in range(4):
        print(f"late ranks N={N} T={T} H={H} forced={forced} {mode} step {step}", flush=True)
        ea, eb = a.step(T), b.step(T)
        assert ea == eb
        got = to_host(a.out_d)
        exp = oracle.reduce_chain(a.pool, ea, T)
        for i in range(L):
            assert np.array_equal(got[i, :T], exp[i]), f"step={step} node={i}"
        _same_words(a, b, T, ea)
    for r in (a, b):
        r.s.check()
        r.s.close()


def test_batches_on_both_sides_of_the_launch_rule():
    """4096 chunks fill the GPU with two-wave workgroups: steps of up to 256
    tokens x 8192 are one launch, the next is a graph of launches. One handle
    crosses the line both ways and its epochs go on."""
    N, H, L, T_max = 2, 8192, 3, 258
    w = synth.Workload(84, "one-launch-or-graph", N, (T_max,), H, L, 1, "uniform")
    pool = synth.payload_pool(84, N, T_max, H, 4, "uniform")
    r = StepRun(w, T_max, pool=pool)
    for tokens in (256, 257, 1, 258, 255):
        print(f"launch rule T={tokens}", flush=True)
        assert r.s.step_plan(tokens) == ((1, 1, 4096) if tokens <= 256 else (L + 2, 1, 4096)) or \
            tokens == 1 and r.s.step_plan(1) == (1, 4, 4096)
        epochs = r.step(tokens)
        got = to_host(r.out_d)
        exp = oracle.reduce_chain(pool, epochs, tokens)
        for i in range(L):
            assert np.array_equal(got[i, :tokens], exp[i]), f"tokens={tokens} node={i}"
    # an eager epoch between steps (odd epoch counts, so the base is set anew)
    out = torch.zeros((257, H), dtype=torch.int16, device=r.pool_d.device)
    r.s.produce(r.pool_d[1], 257)
    r.s.reduce(out, 257)
    assert np.array_equal(to_host(out), oracle.reduce(pool[1][:, :257]))
    epochs = r.step(5)
    exp = oracle.reduce_chain(pool, epochs, 5)
    got = to_host(r.out_d)
    for i in range(L):
        assert np.array_equal(got[i, :5], exp[i]), f"after an eager epoch, node={i}"
    r.s.check()
    r.s.close()


def test_withheld_stamp_in_one_launch_latches():
    w = synth.Workload(85, "one-launch-withheld", 8, (2,), 1024, 6, 1, "normal")
    r = StepRun(w, 2, max_attempts=7)
    r.s.set_injection(inject_table(np.zeros(6), withheld=np.array([0, 0, 4, 0, 0, 0])))
    r.step(2)
    assert r.s.status() == -5
    kind, epoch, chunk, attempts = r.s.error_info()
    assert (kind, epoch, attempts) == (1, 3, 7) and chunk < 4
    log = r.s.read_log()[2, :4]
    assert np.all((log & 0xFFFF) == 7) and np.all((log >> 24) == 4)
    r.s.close()


@pytest.mark.parametrize("N,T,H,L,G,p", [(8, 2, 4104, 5, 1, 0.0), (3, 16, 8192, 4, 2, 0.0),
                                         (4, 17, 8192, 3, 2, 0.0), (7, 5, 3592, 4, 1, 0.0),
                                         (8, 3, 8192, 6, 1, 0.3), (5, 9, 1000, 5, 2, 0.1),
                                         (1, 1, 520, 1, 1, 0.0), (2, 40, 8192, 3, 4, 0.1)])
@pytest.mark.parametrize("mode", ["spec", "ordered"])
def test_epilogue_one_launch_equals_separate_launches(N, T, H, L, G, p, mode):
    w = synth.Workload(87, f"one-launch-epi-{N}-{T}-{H}", N, (T,), H, L, 1, "act", epilogue=True)
    a = StepRun(w, T, validate=mode, fuse_peers=1)
    b = StepRun(w, T, validate=mode, fuse_peers=0, waves_per_group=G, pool=a.pool)
    if p:
        late = synth.delay_table(87, N, 2 * L + 1, p)
        for r in (a, b):
            r.s.set_injection(inject_table(late))
    res = a.res0.copy()
    for step in range(3):
        print(f"epilogue one launch N={N} T={T} H={H} {mode} step {step}", flush=True)
        ea, eb = a.step(T), b.step(T)
        assert ea == eb
        _, r_list, y_list = oracle.reduce_chain(a.pool, ea, T, epilogue=(res, a.weight, w.rms_eps))
        y = to_host(a.y_d)
        for i in range(L):
            assert ulp_distance(y[i], y_list[i]).max() <= 1, f"step={step} node={i}"
        for r in (a, b):
            assert np.array_equal(to_host(r.res_d), r_list[-1]), f"residual, step={step}"
        _same_words(a, b, T, ea)
        res = r_list[-1]
    for r in (a, b):
        r.s.check()
        r.s.close()


def test_epilogue_batches_on_both_sides_of_the_launch_rule():
    """With the epilogue a step is one launch up to a quarter of the GPU's places
    (640 to 1024 chunks by rank count), a graph of launches beyond: one handle
    crosses the line both ways, and an eager epoch follows."""
    N, H, L, T_max = 2, 8192, 4, 66
    w = synth.Workload(88, "one-launch-epi-or-graph", N, (T_max,), H, L, 1, "act", epilogue=True)
    pool = synth.payload_pool(88, N, T_max, H, 5, "act")
    r = StepRun(w, T_max, pool=pool)
    res = r.res0.copy()
    crossed = set()
    for tokens in (40, 66, 1, 64, 65, 33):
        print(f"epilogue launch rule T={tokens}", flush=True)
        launches, _, cap = r.s.step_plan(tokens)
        assert 640 <= cap <= 1024 and launches == (1 if tokens * 16 <= cap else L + 2)
        crossed.add(launches)
        epochs = r.step(tokens)
        _, r_list, y_list = oracle.reduce_chain(pool, epochs, tokens,
                                                epilogue=(res[:tokens], r.weight, w.rms_eps))
        res[:tokens] = r_list[-1]
        assert np.array_equal(to_host(r.res_d), res), tokens
        y = to_host(r.y_d)
        for i in range(L):
            assert ulp_distance(y[i, :tokens], y_list[i]).max() <= 1, (tokens, i)
    assert crossed == {1, L + 2}
    r.s.check()
    r.s.close()


@pytest.mark.parametrize("N", range(1, 9))
@pytest.mark.parametrize("mode", ["spec", "ordered", "none"])
def test_small_steps_are_one_launch(N, mode):
    """The rule itself, from the plan the handle states: 16 two-wave workgroups
    on each of 256 CUs (with the epilogue a quarter of what fits, 640 chunks at
    least), four consumer waves up to 256 chunks; everything else is launches."""
    def plan(tokens, hidden=4096, L=6, table=False, **cfg):
        with S.Sifar(nranks=N, hidden=hidden, max_tokens=tokens, reduces_per_step=L, validate=mode,
                     **cfg) as s:
            if table:
                s.set_injection([0] * L)
            return s.step_plan(tokens)

    assert plan(1) == (1, 4, 4096) and plan(32) == (1, 4, 4096)
    assert plan(33) == (1, 1, 4096) and plan(512) == (1, 1, 4096)
    assert plan(513) == (8, 1, 4096)
    launches, waves, cap = plan(8, 8192, epilogue=1)
    assert (launches, waves) == (1, 4) and 640 <= cap <= 1024
    assert plan(cap // 16, 8192, epilogue=1) == (1, 1, cap)
    assert plan(cap // 16 + 1, 8192, epilogue=1) == (8, 1, cap)
    assert plan(2, 65 * 512, epilogue=1, waves_per_group=2) == (8, 1, 0)  # 65 chunks a token
    assert plan(4, fuse_peers=0) == (13, 1, 0) and plan(4, buffers=1) == (13, 1, 0)
    if mode == "ordered":
        assert plan(4, persistent=1) == (1, 1, 0)
    if mode != "none":
        assert plan(1, table=True) == (1, 1, 4096)


def test_epilogue_steps_of_four_handles_at_once():
    """Four handles' one-launch epilogue steps on four streams: their token
    exchanges wait inside the launches, so all must fit the GPU together."""
    N, T, H, L = 8, 32, 8192, 8
    w = synth.Workload(89, "one-launch-epi-4", N, (T,), H, L, 1, "act", epilogue=True)
    pool = synth.payload_pool(89, N, T, H, 5, "act")
    runs = [StepRun(w, T, pool=pool) for _ in range(4)]
    streams = [torch.cuda.Stream() for _ in runs]
    torch.cuda.synchronize()
    for step in range(6):
        print(f"four handles step {step}", flush=True)
        for r, st in zip(runs, streams):
            r.s.step(T, st)
    torch.cuda.synchronize()
    res = runs[0].res0.copy()
    for step in range(6):
        epochs = range(1 + step * L, 1 + (step + 1) * L)
        _, r_list, _ = oracle.reduce_chain(pool, epochs, T, epilogue=(res, runs[0].weight, w.rms_eps))
        res = r_list[-1]
    for r in runs:
        r.s.check()
        assert np.array_equal(to_host(r.res_d), res)
        r.s.close()


@pytest.mark.parametrize("epilogue", [False, True])
def test_forced_retries_without_a_table(epilogue):
    """Every validation repeated twice, in steps whose chunks have four consumer
    waves: each wave repeats its own, the log counts three."""
    N, T, H, L = 8, 2, 1000, 5
    w = synth.Workload(94, "one-launch-forced", N, (T,), H, L, 1, "act", epilogue=epilogue)
    a = StepRun(w, T, forced_retries=2)
    b = StepRun(w, T, forced_retries=2, fuse_peers=0, pool=a.pool)
    for step in range(2):
        ea, eb = a.step(T), b.step(T)
        assert ea == eb
        _same_words(a, b, T, ea)
        assert np.all((a.s.read_log()[:L, :4] & 0xFFFF) == 3)
        if epilogue:
            assert np.array_equal(to_host(a.res_d), to_host(b.res_d))
        else:
            assert np.array_equal(to_host(a.out_d), to_host(b.out_d))
    for r in (a, b):
        r.s.check()
        r.s.close()
