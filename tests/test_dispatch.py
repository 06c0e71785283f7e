"""Which kernels a batch takes (csrc/dispatch.h), asked on the host."""
import ctypes
import importlib.util
import os

import numpy as np
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
    (2, DSV3, A8, True, "stream_a8"), (5, QWEN3, A8, True, "tiled_a8"),
    # 3 tokens x 8 slots x 16 column blocks: not routed inside, and H is long
    (3, DSV3, A8, True, "tiled_a8"), (4, (4096, 14336, 8, 2), A8, True, "stream_a8"),
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
                    p, routes, _ = eaas._gemm_plan(T, 512, 256, E, k, wdt, gate_up, capacity)
                    assert p != "one_wave" or T <= 32, (T, E, k)
                    assert not routes or T <= 64, (T, E, k)
    assert eaas._gemm_plan(32, 2048, 128, 256, 8, wdt, True, capacity)[:2] == ("one_wave", True)
    assert eaas._gemm_plan(64, 2048, 512, 32, 8, wdt, True, capacity)[:2] == ("few", True)


@pytest.mark.parametrize("wdt", [BF16, FP8, eaas.EAAS_FP8_E4M3_TILED])
def test_self_routing_grids_fit_the_chip(wdt):
    """Groups without rows are not compacted away by a launch that routes
    itself: four-wave workgroups are then at most what the chip holds at once
    (two on each of 256 CUs), so that those with rows cannot pile up."""
    for E in (1, 8, 24, 32, 64, 128, 256, 1024):
        for k in (1, 2, 6, 8):
            for I in (128, 640, 768, 2048, 14336):
                for T in (1, 2, 3, 4, 8, 16, 17, 32, 33, 64):
                    p, routes, _ = eaas._gemm_plan(T, 1024, I, E, k, wdt, True)
                    waves = min(E, T * k) * 2 * I // 32
                    assert not (routes and p == "few") or waves <= 2048, (T, E, k, I)
    assert eaas._gemm_plan(16, 1024, 1024, 32, 8, wdt, True)[:2] == ("few", True)  # 2 048 waves
    assert eaas._gemm_plan(16, *DSV3, wdt, True)[:2] == ("few", False)             # 4 096
    assert eaas._gemm_plan(8, *DSV3, wdt, True)[:2] == ("one_wave", True)


MIXTRAL = (4096, 14336, 8, 2)


def even(rows, E):
    return [rows // E + (e < rows % E) for e in range(E)]


@pytest.mark.parametrize("T,shape,wdt,gate_up,capacity,counts,expect", [
    # a full dynamic batch takes the tiled kernels, a part-filled one streams
    (1920, MIXTRAL, FP8, True, True, even(3840, 8), "tiled"),
    (1920, MIXTRAL, FP8, True, True, even(890, 8), "wide8"),
    (1920, MIXTRAL, FP8, False, True, even(3840, 8), "tiled"),
    (1920, MIXTRAL, FP8, False, True, even(890, 8), "wide4"),
    (2400, MIXTRAL, FP8, False, True, even(890, 8), "wide4"),
    (512, QWEN3, BF16, True, True, even(4096, 128), "few"),
    (768, QWEN3, BF16, True, True, even(6144, 128), "tiled"),
    (768, QWEN3, BF16, True, True, even(3000, 128), "few"),
    # hot experts: further blocks for one in four (bf16, 64 rows) or five (144 rows)
    (512, QWEN3, BF16, True, True, [512] * 4 + even(2048, 124), "few"),
    (512, QWEN3, BF16, True, True, [512] * 5 + even(1536, 123), "tiled"),
    (384, QWEN3, BF16, True, False, [384] * 8 + [0] * 120, "tiled"),
    (256, DSV3, FP8, True, False, even(2048, 32), "wide8"),
    (256, DSV3, FP8, True, False, [145] * 6 + even(1178, 26), "wide8"),
    (256, DSV3, FP8, True, False, [145] * 7 + even(1033, 25), "tiled"),
    # few active experts: the blocks fill the chip no more than once
    (256, DSV3, FP8, True, False, [256] * 8 + [0] * 24, "wide8"),
    (300, DSV3, FP8, True, False, [300] * 8 + [0] * 24, "tiled"),
    (768, QWEN3, FP8, True, True, [600] * 30 + [0] * 98, "tiled"),
    (300, (384, 128, 5, 2), BF16, True, False, [300, 300, 0, 0, 0], "wide4"),
    # no choice where an expert has one block, or further ones are few
    (64, DSV3, FP8, True, False, [64] * 8 + [0] * 24, "few"),
    (144, DSV3, FP8, True, False, [144] * 8 + [0] * 24, "wide8"),
    (480, DSV3, FP8, False, False, even(3840, 32), "tiled")])
def test_rows_choose_the_kernel(T, shape, wdt, gate_up, capacity, counts, expect):
    assert eaas._gemm_plan(T, *shape, wdt, gate_up, capacity, counts)[0] == expect


@pytest.mark.parametrize("wdt", [BF16, FP8, eaas.EAAS_FP8_E4M3_TILED])
@pytest.mark.parametrize("shape", [QWEN3, DSV3, MIXTRAL, (1920, 640, 24, 6), (2048, 512, 256, 1)])
def test_full_and_skewed_batches_are_not_streamed_block_after_block(shape, wdt):
    """Whatever the batch, streaming launches that read an active expert's
    weights more than twice fill the chip no more than once (N a multiple of
    256), and a dynamic batch of the same rows takes the kernels of a plain one
    or streams where that is left to it."""
    H, I, E, k = shape
    if wdt == eaas.EAAS_FP8_E4M3_TILED and H % 256:
        pytest.skip("the tiled layout needs H a multiple of 256")
    for T in (65, 145, 200, 256, 257, 384, 512, 1024, 1920, 4096):
        hot = [T] * min(k, E) + [0] * (E - min(k, E))
        half = [T // 2] * min(2 * k, E) + [0] * (E - min(2 * k, E))
        for counts in (even(T * k, E), hot, half):
            for gate_up, N in ((True, 2 * I), (False, H)):
                if N % 256:
                    continue
                for capacity in (False, True):
                    p = eaas._gemm_plan(T, *shape, wdt, gate_up, capacity, counts)[0]
                    height = {"few": 64, "one_wave": 32, "wide8": 144, "wide4": 144}.get(p)
                    if height is None or (p == "few" and T <= 256 and T * k <= 16 * E):
                        continue
                    active = sum(c > 0 for c in counts)
                    blocks = sum(-(-c // height) for c in counts)
                    cols, slots = {"few": (128, 512), "one_wave": (32, 2048), "wide8": (256, 256),
                                   "wide4": (128, 256)}[p]
                    spare = 4 / 3 if p == "few" and wdt != BF16 else 5 / 4
                    assert blocks <= spare * active or blocks * (N // cols) <= slots, (
                        T, p, gate_up, capacity, counts[:10])


@pytest.mark.parametrize("wdt", [BF16, FP8])
@pytest.mark.parametrize("shape", [QWEN3, DSV3, MIXTRAL, (512, 512, 72, 2), (512, 256, 160, 2)])
def test_a_batch_that_streams_fits_the_streaming_launch(shape, wdt):
    """The streaming launch of a batch whose rows decide has room for no more
    row blocks than a batch that streams can have."""
    H, I, E, k = shape
    rng = np.random.default_rng(E)
    chosen = 0
    for T in (100, 150, 257, 300, 512, 1000, 3000):
        for gate_up in (True, False):
            s = eaas._shape(T, H, I, E, k)
            r = eaas.lib().eaas_internal_gemm_plan(ctypes.byref(s), wdt, 1, int(gate_up), None)
            if not r & 32:
                continue
            room, height = r >> 8, {2: 64, 3: 144, 4: 144}[r & 15]
            for trial in range(300):
                p = rng.dirichlet(np.full(E, 10.0 ** rng.uniform(-2, 2)))
                counts = rng.multinomial(rng.integers(1, T * k + 1), p)
                if trial % 3 == 0:  # blocks that are barely begun
                    counts = np.minimum(counts // height * height + 1, T * k)
                if eaas._gemm_plan(T, *shape, wdt, gate_up, True, counts)[0] == "tiled":
                    continue
                chosen += 1
                assert -(-counts // height).sum() <= room
    assert chosen


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
