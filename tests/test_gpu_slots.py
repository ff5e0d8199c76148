"""GPU check of the capacity slots at the edges of the assignment's forms: one
wave block or four per block, histograms added up row by row or by groups of
running sums, more (rank, expert) columns than threads; against a stable sort of
the GPU's own ids in (rank, token) order.  Bit-exact."""

import numpy as np
import pytest
import torch

import paper_2203_14685_amd as hm
from paper_2203_14685_amd import workloads as wl

from _parity import announce, assert_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.load()
    yield


def reference(ids, E, C):
    S, k = ids.shape
    flat = ids.T.reshape(-1)
    demand = np.bincount(flat, minlength=E)
    order = np.argsort(flat, kind="stable")
    place = np.empty(S * k, dtype=np.int64)
    place[order] = np.arange(S * k) - (np.cumsum(demand) - demand)[flat[order]]
    slots = np.where(place < C, place, -1).reshape(k, S).T
    src = np.full((E, C), -1, dtype=np.int64)
    s, r = np.nonzero(slots >= 0)
    src[ids[s, r], slots[s, r]] = s * k + r
    return slots, np.minimum(demand, C), demand, src


@pytest.mark.parametrize("S,E,k", [
    (1, 1, 1), (63, 64, 2), (65, 130, 4), (4096, 256, 1), (8325, 256, 1),  # 32 K counts, one row more (groups)
    (300, 200, 8), (8000, 1024, 8),                                        # more columns than threads
    (32705, 60, 1), (32833, 64, 1), (33000, 16, 8), (33001, 512, 8),       # four wave blocks per block, ragged
    (128001, 128, 8),                                                      # groups of 64 rows
    (65536, 5, 1), (65600, 5, 1), (65601, 300, 1), (131072, 3, 2), (131073, 3, 2),  # sixteen wave blocks per block
    (50000, 24, 2), (66001, 16, 4), (66001, 13, 5), (33100, 64, 1),                 # 512 threads after group_scan, and not
    (131200, 64, 8), (131200, 65, 8),                                      # 512 columns, and too many for sixteen
    (200, 2, 1), (4000, 1, 1), (2100, 3, 3),                               # many partial sums per column
])
def test_slots(S, E, k):
    announce(f"slots S={S} E={E} k={k}")
    g = torch.Generator(device="cuda")
    g.manual_seed(S + E)
    L = torch.randn((S, E), generator=g, device="cuda")
    L[:, : max(1, E // 16)] += 1.0  # favoured experts overflow their capacity
    for C in (0, max(1, S * k // (2 * E)), S * k // E + 37):
        o = hm.gate(hm.MOE_GATE_TOPK, k, E, C, logits=L, logits_in=True)
        torch.cuda.synchronize()
        slots, counts, demand, src = reference(wl.to_host(o["ids"]), E, C)
        assert_equal(wl.to_host(o["slots"]), slots, "slots")
        assert_equal(wl.to_host(o["counts"]), counts, "counts")
        assert_equal(wl.to_host(o["demand"]), demand, "demand")
        assert_equal(wl.to_host(o["slot_src"]), src, "slot_src")
