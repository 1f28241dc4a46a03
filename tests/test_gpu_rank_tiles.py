"""Ranks at the edges of the score tiles (needs an MI355X).

Rows are small whole numbers, each row times a power of two of its own: every
score is exact in float32, ties with the positive score are frequent, and the
ranks must equal the oracle's without exception.  Entities around the tiles of
128 columns and the blocks of 64, queries around 128 and 256 rows, rows around
the slices of 32 elements, and more queries than one block of 2^18 takes."""

import numpy as np
import pytest

from oracle import pbg_oracle as O
from paper_1903_12287_amd import synth
from tests.test_gpu_rank import _gpu_ranks
from tests.test_gpu_rank_sampled import _gpu_sampled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("op,n,m,d", [
    ("identity", 1, 1, 1),
    ("translation", 63, 127, 32),
    ("identity", 65, 128, 33),
    ("diagonal", 128, 129, 64),
    ("translation", 129, 256, 200),
    ("identity", 1000, 1153, 96),
    ("identity", 70, 262_200, 8),
])
def test_exact_ranks_at_tile_edges(op, n, m, d, sampled):
    rng = synth.rng_for(97 + n + d)
    emb = rng.integers(-3, 4, (n, d)).astype(np.float32)
    # translation adds rows of unlike scales, so its rows share one
    if op != "translation":
        emb *= np.exp2(rng.integers(-30, 31, (n, 1))).astype(np.float32)
    relp = None if op == "identity" else rng.integers(-2, 3, (1, d)).astype(np.float32)
    src, dst = (rng.integers(0, n, m).astype(np.int32) for _ in range(2))
    idx = np.unique(np.r_[0:min(m, 400), max(0, m - 400):m])
    model = O.Model.create(n, 1, 1, d, op, "dot", "softmax", 0.1, [emb.astype(np.float64)],
                           None if relp is None else relp.astype(np.float64))
    if sampled:
        cand = rng.integers(0, n, 2 * n + 1).astype(np.int32)
        got, _, _ = _gpu_sampled(n, 1, d, op, "dot", emb, relp, src, None, dst, cand)
        want = O.rank_sampled(model, src[idx], None, dst[idx], cand)[0]
    else:
        ks, kd = np.r_[src[:300], src[:50]], np.r_[dst[:300], dst[:50]]
        got, _, _ = _gpu_ranks(n, 1, d, op, "dot", emb, relp, src, None, dst, ks, None, kd)
        want = O.rank_eval(model, src[idx], None, dst[idx], ks, None, kd)[0]
    np.testing.assert_array_equal(np.concatenate([got[idx], got[m + idx]]), want)
