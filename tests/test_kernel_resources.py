"""Register budgets of the step kernels, checked at compile time.

A persistent step needs every one of its waves resident at once. The payload
sweep's largest step (N = 8, T = 256, H = 8192: 4096 chunks) fills an MI355X
exactly: 8192 one-wave workgroups, i.e. 8 waves per SIMD, which gfx950 grants
only to kernels of at most 64 VGPRs. Compiling the
device code here (hipcc cross-compiles without a GPU) catches a change that
pushes those kernels past the budget before a GPU run skips or refuses the
step. No GPU is used.

A per-epoch step is one launch while its chunks fit the GPU at once, up to 16
two-wave workgroups per CU: the limit comes from the same registers, and the
launch bounds turn growth into spills rather than into fewer places.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2607_08973_amd import build as B

VGPRS_FOR_8_WAVES_PER_SIMD = 64


def _hipcc():
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return None


@pytest.fixture(scope="module")
def kernel_resources(tmp_path_factory):
    """{mangled kernel name: {"vgpr": n, "spill": n, "sgpr_spill": n, "scratch": bytes}}
    from the device assembly."""
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("isa") / "kernels.s"
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [hipcc, *flags, "--cuda-device-only", "-S", "-I", B.INCLUDE, "-I", B.CSRC,
           os.path.join(B.CSRC, "kernels.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    text = out.read_text()
    found = {}
    # kernel metadata entries: ".name: <sym>" ... ".vgpr_count: n", ".vgpr_spill_count: n"
    for m in re.finditer(r"\.name:\s+(\S+)\n(.*?)(?=\n\s+- \.|\n\s+-\s|\Z)", text, re.S):
        body = m.group(2)
        v = re.search(r"\.vgpr_count:\s+(\d+)", body)
        if v:
            n = lambda key: int((re.search(rf"\.{key}:\s+(\d+)", body) or [0, 0])[1])
            found[m.group(1)] = {"vgpr": int(v.group(1)), "spill": n("vgpr_spill_count"),
                                 "sgpr_spill": n("sgpr_spill_count"),
                                 "scratch": n("private_segment_fixed_size")}
    assert found, "no kernel metadata in the device assembly"
    return found


def _chain(n, epi, prefetch):
    b = lambda x: "1" if x else "0"
    return (f"_ZN5sifar12_GLOBAL__N_112chain_kernelILi{n}ELi1ELb{b(epi)}"
            f"ELb{b(prefetch)}EEEvNS_9ChainArgsE")


def test_largest_steps_fit_eight_waves_per_simd(kernel_resources):
    """The non-prefetching one-wave kernel of a plain N = 8 step stays within
    64 VGPRs (the form init falls back to when a step needs every wave slot of
    the GPU)."""
    name = _chain(8, False, False)
    assert name in kernel_resources, name
    assert kernel_resources[name]["vgpr"] <= VGPRS_FOR_8_WAVES_PER_SIMD, (
        name, kernel_resources[name])


def test_prefetching_kernel_keeps_its_occupancy(kernel_resources):
    """The prefetching one-wave kernel (the llama8b decode step's) holds two
    epochs' sources. At most 80 VGPRs keeps 6 waves per SIMD, enough for
    one-wave steps of up to 3072 chunks (larger handles fall back to the
    non-prefetching form), and it does not spill. (A producer slot wait
    without its short sleep once took it to 109.)"""
    name = _chain(8, False, True)
    assert name in kernel_resources, name
    r = kernel_resources[name]
    assert r["vgpr"] <= 80 and r["spill"] == 0, (name, r)


def _step(n, mode, epi, inject, consumers):
    b = lambda x: "1" if x else "0"
    return (f"_ZN5sifar12_GLOBAL__N_111step_kernelILi{n}ELi{mode}ELb{b(epi)}ELb{b(inject)}"
            f"ELi{consumers}EEEvNS_9ChainArgsE")


@pytest.mark.parametrize("epi,vgprs", [(False, VGPRS_FOR_8_WAVES_PER_SIMD), (True, 96)])
def test_one_launch_steps_keep_their_places(kernel_resources, epi, vgprs):
    """Every one-launch step kernel within the registers of 8 waves per SIMD (5
    with the epilogue), with nothing in scratch memory: the launch rule counts
    on those places, and a spill would be paid in every all-reduce. Kernels
    without an injection table keep their scalars in registers too."""
    for n in range(1, 9):
        for mode in (0, 1, 2):
            for inject, consumers in ((False, 1), (False, 4), (True, 1)):
                name = _step(n, mode, epi, inject, consumers)
                if inject and mode == 2:   # NONE validates nothing: no injection
                    assert name not in kernel_resources
                    continue
                r = kernel_resources[name]
                assert r["vgpr"] <= vgprs and r["spill"] == 0 and r["scratch"] == 0, (name, r)
                if not inject:
                    assert r["sgpr_spill"] == 0, (name, r)


@pytest.mark.parametrize("epi,bound", [(False, 48), (True, 24)])
def test_injecting_steps_spill_few_scalars(kernel_resources, epi, bound):
    """The kernels that know the injection table exceed their scalar registers
    (78 at 8 waves per SIMD); a descriptor per late rank once took them to 55,
    with the epilogue 45."""
    for n in range(1, 9):
        for mode in (0, 1):
            name = _step(n, mode, epi, True, 1)
            assert kernel_resources[name]["sgpr_spill"] <= bound, (name, kernel_resources[name])


def test_persistent_epilogue_keeps_its_places(kernel_resources):
    """Persistent epilogue steps: 5 waves per SIMD (2560 chunks), no spills."""
    for n in range(1, 9):
        r = kernel_resources[_chain(n, True, True)]
        assert r["vgpr"] <= 96 and r["spill"] == 0 and r["scratch"] == 0, (n, r)


def test_one_launch_all_reduce_keeps_its_places(kernel_resources):
    names = [k for k in kernel_resources if "once_kernel" in k]
    assert len(names) == 8
    for name in names:
        r = kernel_resources[name]
        assert r["vgpr"] <= VGPRS_FOR_8_WAVES_PER_SIMD, (name, r)
        assert r["spill"] == 0 and r["sgpr_spill"] == 0 and r["scratch"] == 0, (name, r)
