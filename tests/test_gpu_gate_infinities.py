"""Infinite logits and gradients where a result is defined: a kTop1 group's best
logit counts exp(0) = 1 in its own sum, and dW and dx of an infinite dL are
infinite, not NaN."""

import numpy as np
import pytest
import torch

import paper_2203_14685_amd as hm
from paper_2203_14685_amd import workloads as wl

from _parity import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.load()
    yield


@pytest.mark.parametrize("E,k", [(12, 3), (60, 4), (256, 8), (300, 2), (1023, 3), (5, 5)])
def test_ktop1_on_given_logits(E, k):
    """One +inf per group, and where a group is one expert -inf too."""
    announce(f"kTop1 infinities, given logits E={E} k={k}")
    S, G = 100, E // k
    rng = np.random.default_rng(E)
    L = rng.standard_normal((S, E)).astype(np.float32)
    best = rng.integers(0, G, (S, k)) + np.arange(k) * G
    np.put_along_axis(L, best, np.inf, axis=1)
    if G == 1:
        L[::2] = -np.inf
    g = hm.gate(hm.MOE_GATE_KTOP1, k, E, S, logits=wl.to_device(L, "f32"), logits_in=True)
    torch.cuda.synchronize()
    assert np.array_equal(wl.to_host(g["ids"]), best)
    assert (wl.to_host(g["weights"]) == 1.0).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("S,d,E,k", [(70, 264, 60, 4), (70, 2568, 60, 3), (70, 264, 5, 5)])
def test_ktop1_projected(dtype, S, d, E, k):
    """The same through the bias of a projection, in one kernel and with K split."""
    announce(f"kTop1 infinities, projected {dtype} S={S} d={d} E={E} k={k}")
    G = E // k
    best = np.random.default_rng(E).integers(0, G, k) + np.arange(k) * G
    bias = np.zeros(E, dtype=np.float32)
    bias[best] = np.inf if G > 1 else -np.inf
    g = torch.Generator(device="cuda")
    g.manual_seed(E)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((S, d), generator=g, device="cuda").to(dt)
    wg = torch.randn((d, E), generator=g, device="cuda").to(dt)
    o = hm.gate(hm.MOE_GATE_KTOP1, k, E, S, x=x, wg=wg, bias=wl.to_device(bias, "f32"))
    torch.cuda.synchronize()
    assert np.array_equal(wl.to_host(o["ids"]), np.broadcast_to(best, (S, k)))
    assert (wl.to_host(o["weights"]) == 1.0).all()


@pytest.mark.parametrize("dtype,d,E", [("bf16", 264, 60), ("bf16", 136, 17), ("bf16", 520, 256), ("f32", 260, 60)])
def test_gate_gradient_of_infinite_dlogits(dtype, d, E):
    """A weight gradient that overflows the temperature's division: dW and dx are
    what IEEE sums of the products with the dL that the call reports give."""
    announce(f"gate bwd infinities {dtype} d={d} E={E}")
    S, k = 100, 1
    g = torch.Generator(device="cuda")
    g.manual_seed(E)
    L = torch.randn((S, E), generator=g, device="cuda")
    L[7] = -200.0  # all the probability on two experts: the others' gradient is finite
    L[7, :2] = 0.0
    ids = torch.argmax(L, dim=1, keepdim=True).to(torch.int32)
    dw = torch.randn((S, k), generator=g, device="cuda")
    dw[7] = 3.0e38
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((S, d), generator=g, device="cuda").to(dt)
    x[x == 0] = 1.0
    wg = torch.randn((d, E), generator=g, device="cuda").to(dt)
    wg[wg == 0] = 1.0
    wg[:, 1] = -wg[:, 0]  # both infinities of a row of dx have one sign
    p = hm.gate_bwd_params(S, d, E, k, 0, 0, hm.MOE_BF16 if dtype == "bf16" else hm.MOE_F32, 0, 0.0, 0.125)
    ws = torch.empty((hm.moe_gate_bwd_workspace_size(p),), dtype=torch.uint8, device="cuda")
    dl, dx, dwg, db = torch.empty_like(L), torch.empty_like(x), torch.empty((d, E), device="cuda"), torch.empty((E,), device="cuda")
    hm.moe_gate_bwd(p, x, wg, L, ids, dw, dl, dx, dwg, db, None, ws)
    torch.cuda.synchronize()
    dl, x, wg, dx, dwg = (t.cpu().double() for t in (dl, x, wg, dx, dwg))
    assert torch.isinf(dl).sum() == 2 and not torch.isnan(dl).any()
    for got, want in ((dwg, x.t() @ dl), (dx, dl @ wg.t())):
        inf = torch.isinf(want)
        assert inf.any() and not torch.isnan(want).any()
        assert torch.equal(got[inf], want[inf])
        assert torch.isfinite(got[~inf]).all()
