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
