"""Which kernels a batch takes (csrc/dispatch.h), asked on the host."""
import importlib.util
import os

import pytest

from paper_2509_17863_amd import eaas, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
QWEN3, DSV3 = (2048, 768, 128, 8), (7168, 2048, 32, 8)
BF16, FP8, A8 = eaas.EAAS_BF16, eaas.EAAS_FP8_E4M3, eaas.EAAS_FP8_E4M3_A8


def path(T, shape, wdt, gate_up=True, capacity=False):
    return eaas._gemm_plan(T, *shape, wdt, gate_up, capacity)[0]


@pytest.mark.parametrize("T,shape,wdt,gate_up,expect", [
    (1, DSV3, FP8, True, "one_wave"), (9, DSV3, FP8, True, "few"),
    (9, DSV3, BF16, False, "few"), (256, DSV3, FP8, True, "wide8"),
    (256, DSV3, FP8, False, "tiled"), (8192, QWEN3, BF16, True, "tiled"),
    (4, DSV3, A8, True, "stream_a8"), (5, DSV3, A8, True, "tiled_a8"),
    (16, DSV3, A8, False, "stream_a8"), (17, DSV3, A8, False, "tiled_a8")])
def test_paths(T, shape, wdt, gate_up, expect):
    assert path(T, shape, wdt, gate_up) == expect


@pytest.mark.parametrize("wdt", [BF16, FP8, eaas.EAAS_FP8_E4M3_TILED])
@pytest.mark.parametrize("capacity", [False, True])
def test_a_hot_expert_is_not_walked_in_series(wdt, capacity):
    """The kernels that walk an expert's rows block by block in one workgroup
    (one wave: 32 rows, self-routing: 64) get no batch of more tokens than one
    block holds: with distinct ids per token no expert has more rows."""
    for E in (1, 2, 16, 32, 128, 256, 1024):
        for k in (1, 2, 4, 8, 64):
            for T in (1, 16, 32, 33, 64, 65, 128, 512, 2048):
                for gate_up in (True, False):
                    p, routes = eaas._gemm_plan(T, 512, 256, E, k, wdt, gate_up, capacity)
                    assert p != "one_wave" or T <= 32, (T, E, k)
                    assert not routes or T <= 64, (T, E, k)
    assert eaas._gemm_plan(32, 2048, 128, 256, 8, wdt, True, capacity) == ("one_wave", True)
    assert eaas._gemm_plan(64, 2048, 512, 32, 8, wdt, True, capacity) == ("few", True)


@pytest.mark.parametrize("wdt", [BF16, FP8, eaas.EAAS_FP8_E4M3_TILED])
def test_self_routing_grids_fit_the_chip(wdt):
    """Groups without rows are not compacted away by a launch that routes
    itself: four-wave workgroups are then at most what the chip holds at once
    (two on each of 256 CUs), so that those with rows cannot pile up."""
    for E in (1, 8, 24, 32, 64, 128, 256, 1024):
        for k in (1, 2, 6, 8):
            for I in (128, 640, 768, 2048, 14336):
                for T in (1, 2, 3, 4, 8, 16, 17, 32, 33, 64):
                    p, routes = eaas._gemm_plan(T, 1024, I, E, k, wdt, True)
                    waves = min(E, T * k) * 2 * I // 32
                    assert not (routes and p == "few") or waves <= 2048, (T, E, k, I)
    assert eaas._gemm_plan(16, 1024, 1024, 32, 8, wdt, True) == ("few", True)  # 2 048 waves
    assert eaas._gemm_plan(16, *DSV3, wdt, True) == ("few", False)             # 4 096
    assert eaas._gemm_plan(8, *DSV3, wdt, True) == ("one_wave", True)


def test_a_long_list_of_experts_needs_a_long_k():
    """Row blocks are found 64 active experts at a time, in series."""
    assert path(2048, (1024, 256, 1024, 1), FP8) == "tiled"
    assert path(2048, (4096, 256, 1024, 1), FP8) == "few"
    assert path(512, (4096, 1024, 512, 8), FP8, False) == "few"
    assert path(128, (1024, 256, 1024, 1), FP8) == "few"      # at most 128 active
    assert path(256, QWEN3, BF16, False) == "few"             # K 768, 128 experts
    assert path(64, (256, 128, 8, 2), BF16, False) == "few"   # K 128, 8 experts


def test_rejected_shapes_have_no_plan():
    for H, wdt in ((100, BF16), (384, A8), (384, eaas.EAAS_FP8_E4M3_TILED)):
        with pytest.raises(eaas.EaasError):
            eaas._gemm_plan(4, H, 128, 8, 2, wdt, True)


def test_bench_names_the_kernel_of_the_librarys_own_rule():
    """bench.py keeps no copy of the dispatch limits: one token either side of
    every change of path, its name follows the library's."""
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    kernel = {"one_wave": "stream_kernel", "few": "shared_kernel", "wide8": "shared_kernel",
              "wide4": "shared_kernel", "tiled_a8": "w8a8_kernel", "stream_a8": "stream_a8_kernel"}
    for shape in (QWEN3, DSV3, tuple(getattr(synth.WORKLOADS["tiny"], a) for a in "HIEk")):
        for wdt, mode in ((BF16, {"wdtype": "bf16"}), (FP8, {"wdtype": "fp8"}),
                          (A8, {"wdtype": "fp8", "act8": True})):
            last = None
            for T in range(1, 1200):
                p = path(T, shape, wdt)
                if p == last:
                    continue
                for t, q in ((T - 1, last), (T, p)):
                    if q is None:
                        continue
                    H, I, E, k = shape
                    name = bench.gate_up_kernel_name(dict(T=t, H=H, I=I, E=E, k=k, **mode))
                    want = kernel.get(q, "dma_kernel" if wdt == FP8 else "pp_kernel")
                    assert f"grouped_gemm_{want}" in name, (shape, wdt, t, q, name)
                last = p
