"""The gate's optional logits output: asking for it changes nothing else, on every
way a projection takes to its selection (one kernel, K split over blocks, and
logits in memory past 256 experts or with W not 16-byte aligned), with and
without noise and a temperature, for moe_gate and moe_gate_noalloc."""

import math

import numpy as np
import pytest
import torch

import paper_2203_14685_amd as hm
from paper_2203_14685_amd import workloads as wl

from _parity import announce, check_gate

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.load()
    yield


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,k,E,groups", [
    (0, 5, 5, 0), (1, 3, 15, 0), (0, 4, 32, 0), (0, 8, 60, 0), (1, 4, 60, 0), (3, 3, 60, 6),
    (0, 2, 256, 0), (1, 8, 256, 0), (3, 2, 256, 4),
    (0, 2, 257, 0), (1, 1, 257, 0), (3, 5, 257, 1),
    (0, 1, 512, 0), (1, 2, 512, 0), (3, 4, 512, 8),
    (0, 8, 1024, 0), (1, 8, 1024, 0), (3, 8, 1024, 4),
])
@pytest.mark.parametrize("d,wofs", [(264, 0), (264, 1), (40, 1), (2568, 0)])  # wofs: elements W is off its alignment by
def test_logits_output_changes_nothing(dtype, kind, k, E, groups, d, wofs):
    S, C = 130, int(math.ceil(0.9 * k * 130 / E))
    rng = np.random.default_rng(E + k)
    w = dict(kind=0, k=k, normalize=0, dtype=dtype, S=S, d=d, E=E, cf=1.0, hot_experts=1, hot_bias=0.5)
    inp = wl.make_inputs(w, seed=E + kind)
    x, bias = wl.to_device(inp["x"], dtype), wl.to_device(inp["bias"], "f32")
    wg = torch.empty((d * E + 16,), dtype=x.dtype, device="cuda")[wofs:wofs + d * E].view(d, E)
    wg.copy_(wl.to_device(inp["wg"], dtype))
    noise = rng.gumbel(size=(S, E)).astype(np.float32)
    for tau in (0.0, 0.5):
        normalize = int(kind != 1 and tau > 0)
        announce(f"logits output {dtype} kind={kind} k={k} E={E} groups={groups} d={d} wofs={wofs} tau={tau}")
        p = hm.gate_params(S, d, E, k, C, kind, normalize, 0, hm.MOE_BF16 if dtype == "bf16" else hm.MOE_F32, 0, groups, tau)
        nz = wl.to_device(noise, "f32") if tau else None
        runs = {}
        for noalloc in (False, True):
            for want in (True, False):
                i32 = lambda *sh: torch.full(sh, -3, dtype=torch.int32, device="cuda")
                o = dict(logits=torch.zeros((S, E), device="cuda") if want else None, ids=i32(S, k), slots=i32(S, k),
                         weights=torch.zeros((S, k), device="cuda"), counts=i32(E), demand=i32(E), slot_src=i32(E, C))
                args = (p, x, wg, bias, None, nz, None, *o.values())
                if noalloc:
                    hm.moe_gate_noalloc(*args)
                else:
                    hm.moe_gate(*args, torch.empty((hm.moe_gate_workspace_size(p),), dtype=torch.uint8, device="cuda"))
                torch.cuda.synchronize()
                runs[noalloc, want] = {key: wl.to_host(v) for key, v in o.items() if v is not None}
        full = runs[False, True]
        for r in runs.values():
            for key in r:
                assert np.array_equal(r[key], full[key]), key
        check_gate(w, inp, full, E, k, C, kind, normalize, groups=groups, noise=noise if tau else None, temperature=tau)
