"""pbg_score_edges after calls that failed: the id check's flags outlive a call,
so one call's verdict must not reach the next."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import pbg_oracle as O
from paper_1903_12287_amd import pbg
from tests.pbg_cases import GpuModel, make_problem, oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op,R,m", [("translation", 3, 1), ("diagonal", 3, 4001), ("linear", 2, 300)])
def test_calls_behind_failed_ones(op, R, m):
    pb = make_problem(op, "dot", "ranking", n=60, R=R, d=16, m=m)
    gm = GpuModel(pb)
    lib = ctypes.CDLL(pbg.LIB_PATH)   # and the HIP runtime it is linked against
    want = O.score_edges(oracle_model(pb), 0, 0, pb.src, pb.rel_ids, pb.dst)
    out = torch.empty(m, dtype=torch.float32, device="cuda")

    def scores_are_right():
        out.fill_(-1.0)
        pbg.pbg_score_edges(gm.ctx, 0, 0, gm.src, gm.rel_ids, gm.dst, out)
        assert np.max(np.abs(out.cpu().numpy() - want)) <= 1e-5 * max(1.0, float(np.max(np.abs(want))))

    try:
        scores_are_right()
        for arg, word in ((0, 1), (1, 4), (2, 2)):   # source, relation, destination; several bad ids at once
            args = [gm.src.clone(), gm.rel_ids.clone(), gm.dst.clone()]
            args[arg][m // 2:] = 60
            out.fill_(-1.0)
            with pytest.raises(pbg.PbgError, match=f"flags {word}"):
                pbg.pbg_score_edges(gm.ctx, 0, 0, *args, out)
            assert bool((out == -1.0).all())   # nothing is written
            scores_are_right()
            # an error that is pending in the runtime ends the call before its verdict is read
            assert lib.hipSetDevice(9999) != 0
            with pytest.raises(pbg.PbgError):
                pbg.pbg_score_edges(gm.ctx, 0, 0, *args, out)
            scores_are_right()
    finally:
        gm.close()
