"""GPU parity of dispatch, combine and their gradients at row lengths of every
unrolling of the choice-major kernels (1 to 8 chunks per lane and step, one or
more steps) and of token rows that take whole waves, against the oracle."""

import numpy as np
import pytest
import torch

import paper_2203_14685_amd as hm
from paper_2203_14685_amd import workloads as wl

from _parity import announce, check_layout_ops, gpu_gate

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.load()
    yield


# chunks of 16 bytes per row: 1, 63, 65, 128, 129, 175, 257, 305, 384, 389, 511, 513, 705, 1025
@pytest.mark.parametrize("S,nch", [(77, n) for n in (1, 63, 65, 128, 129, 175, 257, 305, 384, 389, 511, 513, 705, 1025)] + [
    # whole waves per token row from 1024 rows on (at k = 1 where a block holds one row)
    (1023, 175), (1024, 103), (1024, 175), (1024, 257), (1030, 389)])
@pytest.mark.parametrize("dtype,k", [("bf16", 2), ("f32", 3), ("bf16", 1)])
def test_row_lengths(S, nch, dtype, k):
    E = 6
    d = nch * (8 if dtype == "bf16" else 4)
    C = (20 if k == 1 else 11 * k) * S // 77  # drops and empty slots
    announce(f"layout rows S={S} nch={nch} {dtype} k={k}")
    rng = np.random.default_rng(nch + k)
    L = rng.standard_normal((S, E)).astype(np.float32)
    L[:, 0] += 1.0
    g = gpu_gate(dict(dtype="f32"), None, E, k, C, 0, 1, logits=L)
    check_layout_ops(dict(dtype=dtype), wl.make_rows((S, d), dtype, nch), g["ids"], g["slots"], g["weights"],
                     g["slot_src"], E, C, k, seed=nch)
