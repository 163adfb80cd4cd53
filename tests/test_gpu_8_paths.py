"""GPU parity of the paths a call is sent down by its sizes, at the sizes where each begins and ends.
Bit-exact against the CPU oracle, through the C ABI."""

import numpy as np
import pytest

from efs_gpu import Case, announce, assert_f32_equal, dev
from oracle import efsparse_oracle as O

pytestmark = pytest.mark.gpu


def _messages(d, counts, seed):
    """Per worker counts[w] ascending distinct indices crowded into the first 1024 elements, the rest of
    each message after them, and values from denormals to the largest, signed zeros among them."""
    rng = np.random.default_rng(seed)
    W, K = len(counts), max(counts) + 37
    idx = np.empty((W, K), np.uint32)
    for w, n in enumerate(counts):
        idx[w, :n] = np.sort(rng.choice(1024, size=n, replace=False))
        idx[w, n:] = 1024 + np.sort(rng.choice(d - 1024, size=K - n, replace=False))
    val = (rng.standard_normal((W, K)) * 10.0 ** rng.uniform(-44, 37, (W, K))).astype(np.float32)
    val[rng.random((W, K)) < 0.1] = -0.0
    val[rng.random((W, K)) < 0.3] = np.float32(2.0 ** -149) * rng.integers(-9, 9)
    return idx, val


# entries of the first tile: one chunk of 64 less, exactly, more; marks on both sides of a chunk's edge;
# the packed form's most (4096) and one over; more workers than one group holds
@pytest.mark.parametrize("counts", [[1], [63], [64, 1], [65, 64, 63], [32, 32, 1], [0, 5, 0, 60, 1], [256] * 16,
                                    [256] * 15 + [257], [1024] * 5, [3] * 64, [2] * 65, [40, 0, 90] * 44],
                         ids=lambda c: f"{sum(c)}x{len(c)}")
def test_sparse_aggregate_tile_entries(counts):
    import paper_2009_09271_amd as E
    import torch
    announce("sparse aggregate tile", sum(counts), len(counts))
    d, W = 20011, len(counts)
    idx, val = _messages(d, counts, sum(counts) + W)
    K = idx.shape[1]
    c = Case([0, d], (K + 0.25) / d)
    assert c.K == K
    out = torch.empty(d, dtype=torch.float32, device="cuda")
    for average in (True, False):
        E.decompress_aggregate(c.L, E.EF_MSG_SPARSE, W, dev(idx.view(np.int32)), dev(val), out,
                               c.L.workspace(E.EF_OP_AGG_SPARSE, W), average)
        assert_f32_equal(out, O.decompress_aggregate_sparse(d, idx, val, average), f"average={average}")
