"""Per-epoch steps as graphs of launches with the peers one epoch ahead (a
producer plane in each reduction's launch), on the fallback library: the form
that steps of more chunks than fit the GPU at once take, at the sizes the
one-launch step's tests use. The scenarios are those tests': waves per
workgroup with idle waves, late ranks, forced retries, every validation mode
and rank count, the epilogue's exchange."""
from __future__ import annotations

import pytest

import test_gpu_epilogue_widths as widths
import test_gpu_parity as parity
import test_gpu_step_one_launch as one

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("fallbacks")]


@pytest.mark.parametrize("G", [2, 8, 16])
@pytest.mark.parametrize("mode", ["spec", "ordered"])
def test_multiwave_groups(G, mode):
    parity.test_graph_steps_multiwave_groups(G, mode)


@pytest.mark.parametrize("order", ["spec", "ordered"])
@pytest.mark.parametrize("forced", [0, 2])
def test_stale_injection(order, forced):
    parity.test_stale_injection_deterministic(order, forced, 1)


@pytest.mark.parametrize("mode", ["spec", "ordered", "none"])
def test_llama_decode_steps(mode):
    parity.test_graph_llama_decode_steps(mode, 1)


@pytest.mark.parametrize("T,G", [(1, 1), (8, 4), (32, 16)])
def test_epilogue_moe_chain(T, G):
    parity.test_epilogue_moe_chain(T, G, 1)


@pytest.mark.parametrize("H,G", [(8, 1), (520, 1), (16 * 512 + 8, 2), (33 * 512 - 8, 1), (64 * 512, 16)])
def test_epilogue_exchange_widths(H, G):
    widths.test_epilogue_exchange_widths(H, 0, G, 1)


@pytest.mark.parametrize("mode", ["spec", "ordered", "none"])
@pytest.mark.parametrize("N,T,H,L,G", [(6, 37, 3592, 3, 2), (1, 1, 8, 1, 1), (5, 7, 3896, 5, 16),
                                       (7, 9, 4608, 7, 4)])
def test_equals_separate_launches(N, T, H, L, G, mode):
    one.test_one_launch_equals_separate_launches(N, T, H, L, G, mode)


@pytest.mark.parametrize("mode", ["spec", "ordered"])
@pytest.mark.parametrize("N,T,H,forced", [(8, 2, 4096, 0), (3, 3, 1000, 2)])
def test_late_ranks(N, T, H, forced, mode):
    one.test_late_ranks_catch_up_the_same(N, T, H, forced, mode)


@pytest.mark.parametrize("mode", ["spec", "ordered"])
@pytest.mark.parametrize("N,T,H,L,G,p", [(4, 17, 8192, 3, 2, 0.0), (8, 3, 8192, 6, 1, 0.3),
                                         (5, 9, 1000, 5, 2, 0.1)])
def test_epilogue_equals_separate_launches(N, T, H, L, G, p, mode):
    one.test_epilogue_one_launch_equals_separate_launches(N, T, H, L, G, p, mode)


def test_withheld_stamp_latches():
    one.test_withheld_stamp_in_one_launch_latches()
