"""GPU parity of the tiled projections (any expert count up to 256, any row
length; K split over blocks for small batches) and of the selection on logits in
memory, at the edges of their tiles, stages and K ranges.  The oracle checks
integers bit for bit on the GPU's own logits, logits within 1e-5 of the sum of
|terms| (tests/_parity.py)."""

import math

import numpy as np
import pytest
import torch

import paper_2203_14685_amd as hm
from paper_2203_14685_amd import workloads as wl

from _parity import announce, check_gate, gpu_gate

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.load()
    yield


def _inputs(dtype, S, d, E, k, kind, normalize, bias, seed):
    w = dict(kind=0, k=k, normalize=normalize, dtype=dtype, S=S, d=d, E=E, cf=1.0)
    if bias:
        w.update(hot_experts=1, hot_bias=0.5)
    return w, wl.make_inputs(w, seed=seed)


CASES = [
    # (dtype, S, d, E, k, kind, normalize, groups, tau)
    # expert tiles: one below, at and above each tile count; rows of W that are
    # whole 16-byte pieces, pairs only, and odd
    ("bf16", 65, 264, 1, 1, 0, 0, 0, 0.0), ("bf16", 64, 72, 15, 3, 0, 1, 0, 0.0), ("bf16", 63, 128, 17, 2, 0, 0, 0, 0.5),
    ("bf16", 130, 136, 33, 8, 0, 1, 0, 0.0), ("bf16", 70, 256, 50, 5, 1, 0, 0, 0.0), ("bf16", 1, 8, 63, 7, 1, 0, 0, 0.0),
    ("bf16", 200, 520, 65, 4, 0, 1, 0, 0.0), ("bf16", 66, 384, 96, 6, 3, 1, 4, 0.5), ("bf16", 129, 1032, 97, 1, 0, 0, 0, 0.0),
    ("bf16", 64, 1024, 130, 2, 3, 0, 2, 0.0), ("bf16", 300, 200, 192, 8, 1, 0, 0, 0.0), ("bf16", 65, 1400, 193, 8, 0, 0, 0, 0.0),
    ("bf16", 100, 640, 256, 8, 0, 1, 0, 0.0), ("bf16", 77, 264, 255, 3, 3, 1, 5, 0.0),
    ("f32", 65, 260, 1, 1, 0, 0, 0, 0.0), ("f32", 64, 4, 15, 3, 0, 1, 0, 0.0), ("f32", 63, 132, 18, 2, 1, 0, 0, 0.5),
    ("f32", 130, 68, 33, 8, 0, 1, 0, 0.0), ("f32", 66, 516, 66, 6, 3, 1, 3, 0.0), ("f32", 129, 1028, 129, 1, 0, 0, 0, 0.0),
    ("f32", 300, 200, 192, 8, 1, 0, 0, 0.0), ("f32", 65, 300, 195, 5, 0, 0, 0, 0.5), ("f32", 100, 640, 256, 8, 0, 1, 0, 0.0),
    # K ranges: two and more, the last one ragged, fewer columns than a stage in it
    ("bf16", 40, 520, 24, 2, 0, 1, 0, 0.0), ("bf16", 1000, 2568, 60, 3, 3, 1, 6, 0.5), ("bf16", 7000, 1288, 100, 4, 1, 0, 0, 0.0),
    ("bf16", 2, 6152, 256, 8, 0, 0, 0, 0.0), ("f32", 40, 516, 8, 1, 0, 0, 0, 0.0), ("f32", 1000, 2052, 63, 3, 3, 0, 7, 0.5),
    ("f32", 8000, 516, 40, 2, 0, 1, 0, 0.0),
    # one range, more blocks than CUs
    ("bf16", 20000, 264, 60, 2, 0, 1, 0, 0.0), ("f32", 20000, 132, 20, 2, 0, 0, 0, 0.0),
    # two blocks per CU: from 257 wave blocks past 48 experts, from 513 up to 48
    ("bf16", 16385, 8, 49, 2, 0, 0, 0, 0.0), ("bf16", 16400, 200, 64, 4, 1, 0, 0, 0.5), ("bf16", 16385, 712, 65, 3, 0, 1, 0, 0.0),
    ("bf16", 16400, 136, 96, 8, 3, 1, 4, 0.0), ("bf16", 16449, 72, 97, 1, 0, 0, 0, 0.0), ("bf16", 16385, 264, 128, 8, 0, 0, 0, 0.0),
    ("bf16", 32769, 136, 16, 2, 0, 1, 0, 0.0), ("bf16", 32769, 72, 31, 1, 0, 0, 0, 0.5), ("bf16", 32833, 328, 48, 3, 1, 0, 0, 0.0),
    ("bf16", 32769, 3080, 20, 2, 0, 0, 0, 0.0), ("bf16", 16385, 520, 250, 2, 0, 0, 0, 0.0),
]


@pytest.mark.parametrize("dtype,S,d,E,k,kind,normalize,groups,tau", CASES)
def test_tiled_projection(dtype, S, d, E, k, kind, normalize, groups, tau):
    announce(f"tiled projection {dtype} S={S} d={d} E={E} k={k} kind={kind} groups={groups} tau={tau}")
    w, inp = _inputs(dtype, S, d, E, k, kind, normalize, E % 2 == 1, seed=S + E)
    noise = np.random.default_rng(E).standard_normal((S, E)).astype(np.float32) if tau else None
    C = int(math.ceil(1.1 * k * S / E))
    g = gpu_gate(w, inp, E, k, C, kind, normalize, groups=groups, noise=noise, temperature=tau)
    check_gate(w, inp, g, E, k, C, kind, normalize, groups=groups, noise=noise, temperature=tau)


@pytest.mark.parametrize("dtype,S,d,E", [("bf16", 300, 2568, 60), ("f32", 300, 2052, 60), ("bf16", 100, 4096, 256),
                                         ("f32", 65, 1024, 16)])
def test_split_and_one_block_give_the_same_logits(dtype, S, d, E):
    """A workspace with only the histogram makes one block take every K range of
    its tokens: bitwise the outputs of the split projection, as is the gate that
    runs in the library's scratch."""
    k, C = 2, S
    announce(f"split against one block {dtype} S={S} d={d} E={E}")
    w, inp = _inputs(dtype, S, d, E, k, 0, 0, True, seed=E)
    x, wg, bias = wl.to_device(inp["x"], dtype), wl.to_device(inp["wg"], dtype), wl.to_device(inp["bias"], "f32")
    p = hm.gate_params(S, d, E, k, C, 0, 0, 0, hm.MOE_BF16 if dtype == "bf16" else hm.MOE_F32, 0)
    full = hm.moe_gate_workspace_size(p)
    hist = 4 * k * E * ((S + 63) // 64)
    assert full > hist
    runs = []
    for size in (full, hist, None):
        i32 = lambda *sh: torch.full(sh, -3, dtype=torch.int32, device="cuda")
        o = dict(logits=torch.zeros((S, E), device="cuda"), ids=i32(S, k), slots=i32(S, k),
                 weights=torch.zeros((S, k), device="cuda"), counts=i32(E), demand=i32(E), slot_src=i32(E, C))
        args = (p, x, wg, bias, None, None, None, *o.values())
        if size is None:
            hm.moe_gate_noalloc(*args)
        else:
            hm.moe_gate(*args, torch.empty((size,), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        runs.append(o)
    for r in runs[1:]:
        for key in ("logits", "ids", "slots", "counts", "demand", "slot_src"):
            assert torch.equal(r[key], runs[0][key]), key
        assert torch.allclose(r["weights"], runs[0]["weights"], rtol=2e-6, atol=0)


@pytest.mark.parametrize("S,more,d,E", [(16384, 1, 712, 64), (16384, 70, 200, 96), (16384, 1, 1032, 125),
                                        (32768, 1, 136, 9), (32768, 100, 328, 48), (32768, 1, 1096, 32)])
def test_short_and_long_stages_give_the_same_logits(S, more, d, E):
    """One wave block more takes the batch to two blocks per CU and half as long
    stages: bitwise the logits of the tokens that both batches hold."""
    announce(f"short against long stages S={S}+{more} d={d} E={E}")
    g = torch.Generator(device="cuda")
    g.manual_seed(E)
    x = torch.randn((S + more, d), generator=g, device="cuda").to(torch.bfloat16)
    wg = (torch.randn((d, E), generator=g, device="cuda") / math.sqrt(d)).to(torch.bfloat16)
    runs = [hm.gate(hm.MOE_GATE_TOPK, 1, E, 8, x=x[:n], wg=wg, want_logits=True)["logits"] for n in (S, S + more)]
    torch.cuda.synchronize()
    assert torch.equal(runs[0], runs[1][:S])


@pytest.mark.parametrize("S,E,k,kind,groups,tau", [
    (64, 32, 2, 0, 0, 0.0), (65, 33, 8, 0, 0, 0.0), (130, 256, 8, 0, 0, 0.5), (100, 257, 3, 0, 0, 0.5), (63, 255, 5, 1, 0, 0.0),
    (200, 1024, 8, 3, 4, 0.25), (1, 7, 7, 0, 0, 0.0), (129, 1023, 3, 1, 0, 0.0),
    # four lanes per token past 32 experts: 257 wave blocks and one fewer, 513 where a row is no whole 16-byte pieces
    (16384, 60, 4, 1, 0, 0.5), (16385, 60, 4, 1, 0, 0.5), (16385, 33, 3, 3, 3, 0.0), (16400, 128, 2, 3, 4, 0.25),
    (16390, 128, 8, 1, 0, 0.0), (32768, 127, 2, 0, 0, 0.0), (32769, 127, 1, 1, 0, 0.0),
])
def test_selection_on_given_logits(S, E, k, kind, groups, tau):
    announce(f"selection S={S} E={E} k={k} kind={kind} groups={groups} tau={tau}")
    rng = np.random.default_rng(S + E)
    L = rng.integers(-2, 3, (S, E)).astype(np.float32)  # many ties, zeros of both signs
    L[rng.random((S, E)) < 0.1] = -0.0
    if E > 8 and kind == 0:
        L[:, E // 2] = -np.inf  # a masked expert
        L[:, 1] = np.finfo(np.float32).min
    noise = rng.standard_normal((S, E)).astype(np.float32) if tau else None
    C = int(math.ceil(0.9 * k * S / E))
    import oracle
    sel = L
    if tau:
        with np.errstate(invalid="ignore", over="ignore"):
            sel = oracle.noisy_logits_f32(L, noise, tau)
    for normalize in ((0, 1) if kind != 1 else (0,)):
        g = gpu_gate(dict(dtype="f32"), None, E, k, C, kind, normalize, logits=L, groups=groups, noise=noise, temperature=tau)
        check_gate(dict(dtype="f32"), None, g, E, k, C, kind, normalize, logits_in=sel, groups=groups)
