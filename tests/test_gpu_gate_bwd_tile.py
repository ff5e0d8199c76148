"""GPU parity of the gate backward's tiled products (fp32, and the bf16 shapes
with expert counts or row lengths that the register-sized kernels do not take)
at the edges of their tiles, token ranges and column blocks, against the oracle
with the bounds of test_gpu_gate_bwd."""

import pytest
import torch

import paper_2203_14685_amd as hm

from _parity import announce
from test_gpu_gate_bwd import run_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.load()
    yield


CASES = [
    # (S, d, E, k, kind, normalize, dtype, aux, accumulate)
    # one below, at and above each expert-tile count; E a multiple of 8, of 4, of
    # 2 and odd; d one 16-byte piece, below, at and past a column block
    (65, 8, 1, 1, 0, 0, "bf16", 0.0, False), (64, 72, 15, 2, 0, 1, "bf16", 0.01, True),
    (63, 264, 17, 3, 0, 0, "bf16", 0.0, True), (300, 256, 33, 1, 0, 0, "bf16", 0.02, False),
    (129, 520, 48, 2, 0, 1, "bf16", 0.0, True), (127, 200, 65, 8, 0, 1, "bf16", 0.0, False),
    (128, 136, 98, 2, 1, 0, "bf16", 0.0, True), (257, 1032, 130, 4, 0, 0, "bf16", 0.01, True),
    (100, 320, 192, 6, 1, 0, "bf16", 0.0, False), (70, 1096, 193, 3, 0, 1, "bf16", 0.0, True),
    (500, 384, 256, 8, 0, 1, "bf16", 0.01, False), (33, 64, 255, 5, 0, 0, "bf16", 0.0, True),
    (31, 4, 1, 1, 0, 0, "f32", 0.0, True), (64, 68, 16, 2, 0, 1, "f32", 0.01, False), (65, 260, 18, 2, 1, 0, "f32", 0.0, True),
    (200, 36, 31, 3, 0, 0, "f32", 0.0, False), (129, 252, 66, 2, 0, 1, "f32", 0.0, True),
    (300, 516, 128, 8, 0, 0, "f32", 0.01, False), (50, 100, 191, 1, 0, 0, "f32", 0.0, True),
    (130, 1028, 256, 8, 0, 1, "f32", 0.0, True),
    # several token ranges with a ragged last one, several passes per dx block
    (9000, 1416, 60, 3, 0, 1, "bf16", 0.0, True), (5000, 2056, 200, 2, 0, 0, "bf16", 0.0, False),
    (9000, 516, 40, 2, 0, 0, "f32", 0.01, True),
]


@pytest.mark.parametrize("S,d,E,k,kind,normalize,dtype,aux,acc", CASES)
def test_tiled_gate_bwd(S, d, E, k, kind, normalize, dtype, aux, acc):
    announce(f"tiled gate bwd S={S} d={d} E={E} k={k} kind={kind} normalize={normalize} {dtype} aux={aux} acc={acc}")
    run_case(S, d, E, k, kind, normalize, dtype, aux, acc, seed=S + E)


def test_unaligned_gradient_rows():
    """A caller's dlogits buffer that is 4-byte but not 16-byte aligned gives
    bitwise the results of an aligned one."""
    announce("tiled gate bwd, dlogits off by one float")
    S, d, E, k = 300, 264, 60, 2
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    L = torch.randn((S, E), generator=g, device="cuda")
    ids = torch.topk(L, k, dim=1).indices.to(torch.int32)
    dw = torch.randn((S, k), generator=g, device="cuda")
    for dtype, code in ((torch.bfloat16, hm.MOE_BF16), (torch.float32, hm.MOE_F32)):
        x = torch.randn((S, d), generator=g, device="cuda").to(dtype)
        wg = torch.randn((d, E), generator=g, device="cuda").to(dtype)
        p = hm.gate_bwd_params(S, d, E, k, 0, 1, code)
        ws = torch.empty((hm.moe_gate_bwd_workspace_size(p),), dtype=torch.uint8, device="cuda")
        runs = []
        for off in (0, 1):
            dl = torch.empty((S * E + 4,), device="cuda")[off:off + S * E].view(S, E)
            dx, dwg, db = torch.empty_like(x), torch.empty((d, E), device="cuda"), torch.empty((E,), device="cuda")
            hm.moe_gate_bwd(p, x, wg, L, ids, dw, dl, dx, dwg, db, None, ws)
            torch.cuda.synchronize()
            runs.append((dl.clone(), dx, dwg, db))
        for a, b in zip(*runs):
            assert torch.equal(a, b)
