"""The streaming GEMM kernels of decode-sized batches (a few rows per expert):
row counts at the edges of their 16-row blocks and of their 64- and 144-row
tiles, more than 64 active experts, N that is no multiple of 256, and K of one
tile, an odd number of 128-channel blocks and several ring lengths.

Against the oracle, and bit for bit against the same tokens inside a batch
large enough for the tiled kernels (a token's result does not depend on the
batch around it); the tests ask the library's dispatch that they run what they
name.
"""
import numpy as np
import pytest
import torch

from oracle import eaas_oracle as O
from paper_2509_17863_amd import eaas, synth
from paper_2509_17863_amd.device_io import to_device

pytestmark = pytest.mark.gpu
TOL = 2e-2

# rows per expert; the rest of the E experts stay empty.  "sparse" and "shared"
# take 64-row blocks, the first with few rows per expert and more than 64 active
# ones, and "wide" has enough for 144-row blocks (with 64 experts and I 384, more
# 128-row weight tiles than CUs).
EDGES = {
    "sparse": (128, [33, 17, 16, 15, 2] + [1] * 68),
    "shared": (100, [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 97, 130, 0, 2] + [3] * 60),
    "one expert": (1, [20]),
    "wide": (64, [143, 144, 145, 288, 289, 96, 97, 112, 113, 128, 129, 1, 16, 17] + [40] * 50),
    "wide, few tiles": (6, [144, 145, 96, 17, 160, 1]),
}


def run(dev, k, wdt):
    T, H = dev["x"].shape
    E, twoI, _ = dev["w_gate_up"].shape
    I = twoI // 2
    ws = eaas.alloc_workspace(T, H, I, E, k, wdt)
    ws.fill_(0xFF)
    out = torch.full((T, H), float("nan"), dtype=torch.float32, device="cuda")
    eaas.eaas_expert_forward(dev["x"], dev["topk_ids"], dev["topk_weights"], dev["w_gate_up"],
                             dev["w_down"], out, ws, dev["w_gate_up_scale"], dev["w_down_scale"],
                             act8=wdt == eaas.EAAS_FP8_E4M3_A8,
                             tiled=wdt == eaas.EAAS_FP8_E4M3_TILED)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("rows", list(EDGES))
@pytest.mark.parametrize("wdtype", ["bf16", "fp8", "tiled"])
@pytest.mark.parametrize("H,I", [(128, 128), (384, 384), (1280, 640), (2048, 128)])
def test_row_counts_and_k_lengths(gpu, rows, wdtype, H, I):
    if wdtype == "tiled" and H % 256:
        pytest.skip("the tiled layout needs H a multiple of 256")
    E, counts = EDGES[rows]
    print(f"few rows: {rows} {wdtype} H={H} I={I} E={E} R={sum(counts)}", flush=True)
    rng = np.random.default_rng(len(counts) + H + I)
    small = rng.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)
    # past 120 slots per expert no streaming kernel runs, but for the down GEMM of
    # an H that is no multiple of 256 (test_the_last_128_rows_of_n has its tiled side)
    fill = 130 * E + 200
    big = np.concatenate([small, rng.integers(0, E, fill).astype(np.int32)])
    d = synth.make_inputs(len(big), H, I, E, 1, 77, wdtype="bf16" if wdtype == "bf16" else "fp8")
    d["topk_ids"] = big[:, None].copy()
    d["topk_weights"] = rng.uniform(0.2, 1.0, (len(big), 1)).astype(np.float32)
    sub = O.sub_batch(d, np.arange(len(small)))
    wdt = {"bf16": eaas.EAAS_BF16, "fp8": eaas.EAAS_FP8_E4M3,
           "tiled": eaas.EAAS_FP8_E4M3_TILED}[wdtype]
    for gate_up in (True, False):
        p = eaas._gemm_plan(len(big), H, I, E, 1, wdt, gate_up)[0]
        assert p == ("wide4" if H % 256 and not gate_up else "tiled")
        p = eaas._gemm_plan(len(small), H, I, E, 1, wdt, gate_up)[0]
        if not rows.startswith("wide"):
            assert p == "few"
        elif gate_up and wdtype != "bf16":
            assert p in ("wide8", "wide4")

    def device(inp):
        dev = to_device(inp)
        if wdtype == "tiled":
            for key, which in (("w_gate_up", eaas.EAAS_GATE_UP), ("w_down", eaas.EAAS_DOWN)):
                t = torch.empty_like(dev[key])
                eaas.eaas_tile_weights_fp8(dev[key], which, H, I, t)
                dev[key] = t
        return dev

    got = run(device(sub), 1, wdt)
    whole = run(device(d), 1, wdt)
    assert np.array_equal(got.view(np.uint32), whole[: len(small)].view(np.uint32))
    ref = O.expert_forward(sub)["out"]
    rms = float(np.sqrt((ref ** 2).mean()))
    assert float(np.abs(got - ref).max()) <= TOL * rms


@pytest.mark.parametrize("T,k,E,counts", [
    (32, 4, 64, [34, 33, 32, 17] + [1] * 12),                   # one wave, 32 rows at a time
    (64, 8, 32, [130, 65, 64, 63, 17, 16, 129, 1] + [3] * 9),   # self-routing, 64 at a time
    (65, 8, 33, [130, 65, 64, 63, 17, 16, 129, 1] + [5] * 7)])  # one token more: row blocks
@pytest.mark.parametrize("wdtype", ["bf16", "fp8"])
def test_repeated_ids_fill_several_row_blocks(gpu, T, k, E, counts, wdtype):
    """A token may name an expert more than once, so an expert of a small batch
    can have more rows than one block: the whole step and the separate entry
    points (which never route inside the GEMM), against the oracle."""
    print(f"repeated ids T={T} k={k} E={E} {wdtype}", flush=True)
    H, I = 384, 128
    rng = np.random.default_rng(T + E)
    ids = np.full(T * k, -1, np.int32)
    slots = rng.permutation(np.repeat(np.arange(len(counts)), counts))
    ids[: len(slots)] = slots
    d = synth.make_inputs(T, H, I, E, min(k, E), 79, wdtype=wdtype)
    d.update(k=k, topk_ids=rng.permutation(ids).reshape(T, k).astype(np.int32),
             topk_weights=rng.uniform(0.2, 1.0, (T, k)).astype(np.float32))
    dev = to_device(d)
    wdt = eaas.EAAS_BF16 if wdtype == "bf16" else eaas.EAAS_FP8_E4M3
    got = run(dev, k, wdt)
    ref = O.expert_forward(d)["out"]
    rms = float(np.sqrt((ref ** 2).mean()))
    assert float(np.abs(got - ref).max()) <= TOL * rms
    r = eaas.alloc_routing(T, k, E)
    ws = eaas.alloc_workspace(T, H, I, E, k, wdt)
    y = torch.zeros((T * k, H), dtype=torch.float32, device="cuda")
    out = torch.empty((T, H), dtype=torch.float32, device="cuda")
    eaas.eaas_route_permute(dev["topk_ids"], E, r, ws, H=H, I=I)
    eaas.eaas_expert_ffn_grouped(dev["x"], r, dev["w_gate_up"], dev["w_down"], y, ws, k,
                                 dev["w_gate_up_scale"], dev["w_down_scale"])
    eaas.eaas_unpermute_combine(y, r, dev["topk_weights"], out, E, I=I)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), got.view(np.uint32))


@pytest.mark.parametrize("T,k,E", [(1, 8, 32), (1, 1, 1), (2, 8, 1024), (64, 8, 128), (63, 5, 24),
                                   (64, 8, 32), (4, 8, 33), (128, 4, 65), (512, 1, 512), (3, 2, 2),
                                   (100, 5, 21), (65, 8, 30), (32, 16, 256), (8, 64, 256)])
@pytest.mark.parametrize("wdtype", ["bf16", "fp8"])
def test_routing_of_small_batches(gpu, T, k, E, wdtype):
    """Up to 512 slots of up to 64 tokens the gate/up launch routes the rows
    itself: the routing arrays it writes (and the step's output) against the
    oracle, with masked and repeated ids.  (More tokens or slots take the
    routing launch.)"""
    print(f"small-batch routing T={T} k={k} E={E} {wdtype}", flush=True)
    H, I, R = 128, 128, T * k
    d = synth.make_inputs(T, H, I, E, min(k, E), 5 * T + E, wdtype=wdtype)
    rng = np.random.default_rng(T + k + E)
    ids = rng.integers(0, E, (T, k)).astype(np.int32)  # repeated ids within a token, too
    ids[rng.random((T, k)) < 0.2] = -1
    ids[rng.random((T, k)) < 0.1] = E
    d.update(k=k, topk_ids=ids, topk_weights=rng.uniform(0.1, 1.0, (T, k)).astype(np.float32))
    dev = to_device(d)
    wdt = eaas.EAAS_BF16 if wdtype == "bf16" else eaas.EAAS_FP8_E4M3
    ws = eaas.alloc_workspace(T, H, I, E, k, wdt)
    ws.fill_(0xFF)
    r = eaas.alloc_routing(T, k, E)
    for t in r.values():
        t.fill_(-7)
    out = torch.full((T, H), float("nan"), dtype=torch.float32, device="cuda")
    eaas.eaas_expert_forward(dev["x"], dev["topk_ids"], dev["topk_weights"], dev["w_gate_up"],
                             dev["w_down"], out, ws, dev["w_gate_up_scale"], dev["w_down_scale"],
                             routing=r)
    torch.cuda.synchronize()
    ref = O.expert_forward(d)
    for key, n in (("counts", E), ("offsets", E + 1), ("perm", R), ("inv", R), ("active", E + 1)):
        assert np.array_equal(r[key].cpu().numpy()[:n], ref["routing"][key]), key
    rms = float(np.sqrt((ref["out"] ** 2).mean()))
    assert float(np.abs(out.cpu().numpy() - ref["out"]).max()) <= TOL * rms + (rms == 0.0)


@pytest.mark.parametrize("T,k,E", [(1, 1, 1), (1, 8, 32), (4, 8, 33), (4, 64, 8), (5, 2, 2),
                                   (16, 8, 24), (15, 8, 1024), (16, 40, 64), (16, 64, 1024)])
@pytest.mark.parametrize("H,I", [(256, 128), (768, 384), (1280, 640), (2048, 1152)])
def test_fp8_activations_of_few_tokens(gpu, T, k, E, H, I):
    """fp8 activations: up to 4 (gate/up) or 16 tokens (down) take the streaming
    kernel, with the routing inside the launch (at most E slots and 256
    workgroups) and outside, one to several 16-row blocks (repeated ids), K of
    1 to 16 tiles and masked ids.
    Bit for bit against the tiled kernel, which takes the same tokens inside a
    batch of 17."""
    if E == 1024 and H * I > 256 * 128:
        pytest.skip("one size is enough for 1024 experts")
    print(f"few rows a8: T={T} k={k} E={E} H={H} I={I}", flush=True)
    rng = np.random.default_rng(T + k + E + H)
    d = synth.make_inputs(17, H, I, E, min(k, E), 78, wdtype="fp8")
    ids = rng.integers(0, E, (17, k)).astype(np.int32)
    ids[rng.random((17, k)) < 0.2] = -1
    d.update(k=k, topk_ids=ids, topk_weights=rng.uniform(0.2, 1.0, (17, k)).astype(np.float32))
    dev = to_device(d)
    whole = run(dev, k, eaas.EAAS_FP8_E4M3_A8)
    few = {key: v[:T].contiguous() if key in ("x", "topk_ids", "topk_weights") else v
           for key, v in dev.items()}
    got = run(few, k, eaas.EAAS_FP8_E4M3_A8)
    assert np.isfinite(got).all()
    assert np.array_equal(got.view(np.uint32), whole[:T].view(np.uint32))


@pytest.mark.parametrize("H,I,E,counts", [
    (1920, 128, 4, [1, 255, 2000, 3744]),    # 7 whole tiles and 128 rows
    (384, 256, 3, [20000, 129, 4900]),       # 1 and 128
    (640, 128, 6, [0, 15000, 257, 0, 96, 97])])
@pytest.mark.parametrize("wdtype", ["bf16", "fp8"])
def test_the_last_128_rows_of_n(gpu, H, I, E, counts, wdtype):
    """N no multiple of 256 in a large batch: the tiled kernel takes N / 256
    tiles and a streaming launch the last 128 rows of the down matrix.  Bit for
    bit against small batches of the same tokens, which stream alone, and
    against the oracle."""
    print(f"last rows of N: {wdtype} H={H} I={I} E={E} R={sum(counts)}", flush=True)
    wdt = eaas.EAAS_BF16 if wdtype == "bf16" else eaas.EAAS_FP8_E4M3
    R = sum(counts)
    assert eaas._gemm_plan(R, H, I, E, 1, wdt, False)[0] == "tiled"
    rng = np.random.default_rng(H)
    d = synth.make_inputs(R, H, I, E, 1, 82, wdtype=wdtype)
    ids = rng.permutation(np.repeat(np.arange(E), counts)).astype(np.int32)
    d["topk_ids"] = ids[:, None].copy()
    d["topk_weights"] = rng.uniform(0.2, 1.0, (R, 1)).astype(np.float32)
    whole = run(to_device(d), 1, wdt)
    # tokens of every expert: the first, the last and some between
    pick = np.unique(np.concatenate([np.flatnonzero(ids == e)[[0, -1]] for e in range(E)
                                     if counts[e]] + [rng.choice(R, 300, replace=False)]))
    sub = O.sub_batch(d, pick)
    assert eaas._gemm_plan(len(pick), H, I, E, 1, wdt, False)[0] == "wide4"
    got = run(to_device(sub), 1, wdt)
    assert np.array_equal(got.view(np.uint32), whole[pick].view(np.uint32))
    ref = O.expert_forward(sub)["out"]
    rms = float(np.sqrt((ref ** 2).mean()))
    assert float(np.abs(whole[pick] - ref).max()) <= TOL * rms


# path: E, k, H, I, capacity, tokens of a batch that streams
CHOICES = {
    "few": (160, 2, 512, 256, 3500, 1200),
    "wide8": (72, 2, 512, 512, 5000, 2000),
    "wide4": (8, 2, 512, 512, 4000, 800),
    "few, N % 256": (160, 2, 384, 256, 3500, 1200),  # (down: few alone)
}


@pytest.mark.parametrize("case", list(CHOICES))
@pytest.mark.parametrize("wdtype", ["bf16", "fp8"])
def test_the_rows_choose_between_streaming_and_tiled(gpu, case, wdtype):
    """A dynamic batch whose capacity leaves the kernel open: part filled it
    streams, full it takes the tiled kernels, and so it does with half the
    experts empty and the rest twice as full.  Each request's rows are bit for
    bit those of the plain step on the same tokens, and near the oracle's."""
    E, k, H, I, cap, some = CHOICES[case]
    path = case.split(",")[0]
    if path == "wide8" and wdtype == "bf16":
        pytest.skip("bf16 gate/up of many tiles takes the tiled kernel")
    print(f"rows choose: {case} {wdtype}", flush=True)
    wdt = eaas.EAAS_BF16 if wdtype == "bf16" else eaas.EAAS_FP8_E4M3
    d = synth.make_inputs(cap, H, I, E, k, 80, wdtype=wdtype)
    for tokens, crowded, expect in ((some, False, path), (cap, False, "tiled"),
                                    (cap, True, "tiled")):
        sub = O.sub_batch(d, np.arange(tokens))
        if crowded:
            sub["topk_ids"] = (sub["topk_ids"] // 2).astype(np.int32)
        counts = np.bincount(sub["topk_ids"].ravel(), minlength=E)
        assert eaas._gemm_plan(cap, H, I, E, k, wdt, True, True, counts)[0] == expect
        dev = to_device(sub)
        whole = run(dev, k, wdt)
        n0 = tokens // 3
        out = torch.full((tokens, H), float("nan"), dtype=torch.float32, device="cuda")
        bufs = [tuple(dev[key][a:b].clone() for key in ("x", "topk_ids", "topk_weights")) + (out[a:b],)
                for a, b in ((0, n0), (n0, tokens))]
        table = eaas.segment_table(bufs)
        sizes = torch.tensor([n0, tokens - n0], dtype=torch.int32, device="cuda")
        ws = eaas.alloc_segments_workspace(cap, H, I, E, k, wdt)
        ws.fill_(0xFF)
        eaas.eaas_expert_forward_segments(table, sizes, 2, cap, k, dev["w_gate_up"],
                                          dev["w_down"], ws, eaas.EAAS_FP32,
                                          dev["w_gate_up_scale"], dev["w_down_scale"])
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.array_equal(got.view(np.uint32), whole.view(np.uint32)), (tokens, crowded)
    ref = O.expert_forward(sub)["out"]
    rms = float(np.sqrt((ref ** 2).mean()))
    assert float(np.abs(got - ref).max()) <= TOL * rms


@pytest.mark.parametrize("case", ["few", "wide4"])
def test_a_captured_step_chooses_on_every_replay(gpu, case):
    """One captured dynamic-batch step serves part-filled and full batches: the
    choice between streaming and tiled kernels is made on the device, again on
    every replay.  Each replay against an eager step with the same counts."""
    E, k, H, I, cap, some = CHOICES[case]
    print(f"captured choice: {case}", flush=True)
    d = synth.make_inputs(cap, H, I, E, k, 83, wdtype="bf16")
    dev = to_device(d)
    out = torch.zeros((cap, H), dtype=torch.float32, device="cuda")
    table = eaas.segment_table([(dev["x"], dev["topk_ids"], dev["topk_weights"], out)])
    sizes = torch.tensor([some], dtype=torch.int32, device="cuda")
    ws = eaas.alloc_segments_workspace(cap, H, I, E, k, eaas.EAAS_BF16)

    def step():
        eaas.eaas_expert_forward_segments(table, sizes, 1, cap, k, dev["w_gate_up"],
                                          dev["w_down"], ws, eaas.EAAS_FP32)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for tokens in (some, cap, some, some // 2, cap):
        counts = np.bincount(d["topk_ids"][:tokens].ravel(), minlength=E)
        assert eaas._gemm_plan(cap, H, I, E, k, eaas.EAAS_BF16, True, True, counts)[0] == (
            "tiled" if tokens == cap else case)
        sizes.fill_(tokens)
        out.zero_()
        step()
        eager = out.clone()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), tokens
        assert out[:tokens].abs().sum(dim=1).min().item() > 0
        assert not out[tokens:].any().item()


@pytest.mark.parametrize("wdtype", ["bf16", "fp8"])
def test_the_rows_choose_in_the_separate_entry_points(gpu, wdtype):
    """eaas_expert_ffn_grouped gets its routing from the caller and makes the
    choice by itself: even routing streams, a quarter of the experts with all the
    rows is tiled (bf16).  Bit for bit the whole step, and near the oracle."""
    T, H, I, E, k = 1500, 512, 256, 160, 2
    print(f"separate entry points choose: {wdtype}", flush=True)
    wdt = eaas.EAAS_BF16 if wdtype == "bf16" else eaas.EAAS_FP8_E4M3
    d = synth.make_inputs(T, H, I, E, k, 84, wdtype=wdtype)
    paths = []
    for crowd in (1, 4):
        d["topk_ids"] = (d["topk_ids"] // crowd).astype(np.int32)
        counts = np.bincount(d["topk_ids"].ravel(), minlength=E)
        path, _, by_rows = eaas._gemm_plan(T, H, I, E, k, wdt, True, False, counts)
        assert by_rows
        paths.append(path)
        dev = to_device(d)
        whole = run(dev, k, wdt)
        r = eaas.alloc_routing(T, k, E)
        n = eaas.eaas_workspace_bytes_for(T, H, I, E, k, wdt, eaas.EAAS_ENTRY_FFN_GROUPED)
        ws = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        wsr = eaas.alloc_workspace(T, H, I, E, k, wdt)
        y = torch.zeros((T * k, H), dtype=torch.float32, device="cuda")
        out = torch.empty((T, H), dtype=torch.float32, device="cuda")
        eaas.eaas_route_permute(dev["topk_ids"], E, r, wsr, H=H, I=I)
        eaas.eaas_expert_ffn_grouped(dev["x"], r, dev["w_gate_up"], dev["w_down"], y, ws[:n], k,
                                     dev["w_gate_up_scale"], dev["w_down_scale"])
        eaas.eaas_unpermute_combine(y, r, dev["topk_weights"], out, E, I=I)
        torch.cuda.synchronize()
        assert torch.all(ws[n:] == 0xA5).item()
        got = out.cpu().numpy()
        assert np.array_equal(got.view(np.uint32), whole.view(np.uint32))
        ref = O.expert_forward(d)["out"]
        rms = float(np.sqrt((ref ** 2).mean()))
        assert float(np.abs(got - ref).max()) <= TOL * rms
    assert paths == ["few", "tiled" if wdtype == "bf16" else "few"]
