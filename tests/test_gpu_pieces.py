"""Contractions on row pieces (float32): one step against the oracle at the
edges of the kernels' tiles: 64-wide wave blocks, 128- and 256-row tiles,
16-column blocks, 32-deep slices and their remainders."""
import numpy as np
import pytest

from oracle import pbg_oracle as O
from tests.pbg_cases import GpuModel, gpu_inspect, make_problem, oracle_model

pytestmark = pytest.mark.gpu

# (C, U, edges, d): full and short chunks on both sides of the tile sizes
# (not d = 1: with cos every gradient is then identically zero and the first
# Adagrad step follows the sign of a rounding error)
SHAPES = [(1, 1, 3, 8), (15, 17, 40, 16), (63, 65, 130, 31), (64, 64, 100, 32), (100, 28, 250, 33),
          (127, 129, 300, 65), (128, 257, 250, 100), (129, 1, 270, 112), (255, 300, 260, 113), (256, 0, 300, 128),
          (257, 100, 600, 130), (300, 511, 310, 225)]


@pytest.mark.parametrize("C,U,m,d", SHAPES)
@pytest.mark.parametrize("op,cmp", [("translation", "cos"), ("translation", "dot"), ("diagonal", "dot")])
def test_ranking_step_at_tile_edges(op, cmp, C, U, m, d):
    """Loss, embeddings and accumulators of one step to 1e-5 (float32 sums
    over at most a few hundred candidates; the relation parameters' sums of
    many such rows to 1e-4)."""
    pb = make_problem(op, cmp, "ranking", R=1 if cmp == "cos" else 3, n=400, m=m, d=d, C=C, U=U, S=4, seed=5)
    gm = GpuModel(pb)
    try:
        gl = gm.train()
        st = gm.state()
    finally:
        gm.close()
    om = oracle_model(pb)
    ol = O.train_bucket(om, pb.i, pb.j, pb.src, pb.rel_ids, pb.dst, pb.C, pb.U, pb.S, pb.lr, pb.seed)
    assert abs(gl - ol) <= 1e-5 * max(1.0, abs(ol))
    for got, want, rel in ((st["G"][0], om.G[0], 1e-5), (st["emb"][0], om.emb[0], 1e-5), (st["rel"], om.rel, 1e-4)):
        assert np.max(np.abs(got - want)) <= rel * max(1.0, float(np.max(np.abs(want)))) + 1e-6


@pytest.mark.parametrize("C,U,m,d", SHAPES + [(40, 30, 100, 400)])
@pytest.mark.parametrize("op,cmp,loss", [("translation", "dot", "logistic"), ("diagonal", "cos", "softmax"),
                                         ("diagonal", "dot", "softmax"), ("translation", "cos", "logistic")])
def test_value_loss_step_at_tile_edges(op, cmp, loss, C, U, m, d):
    """As above for the losses whose dS is a float32 matrix.  Embeddings and
    relations to 1e-4: the first Adagrad step is lr g / |g|, so an error of
    K 2^-24 of a row's absolute sum (K up to 800 terms) counts lr K 2^-24 A / |g|
    = 5e-6 A / |g|, and the smooth losses' rows cancel to A / |g| of about 20."""
    pb = make_problem(op, cmp, loss, R=1 if cmp == "cos" else 3, n=400, m=m, d=d, C=C, U=U, S=4, seed=5)
    gm = GpuModel(pb)
    try:
        gl = gm.train()
        st = gm.state()
    finally:
        gm.close()
    om = oracle_model(pb)
    ol = O.train_bucket(om, pb.i, pb.j, pb.src, pb.rel_ids, pb.dst, pb.C, pb.U, pb.S, pb.lr, pb.seed)
    assert abs(gl - ol) <= 1e-5 * max(1.0, abs(ol))
    for got, want, rel in ((st["G"][0], om.G[0], 1e-5), (st["emb"][0], om.emb[0], 1e-4), (st["rel"], om.rel, 1e-4)):
        assert np.max(np.abs(got - want)) <= rel * max(1.0, float(np.max(np.abs(want)))) + 1e-6


@pytest.mark.parametrize("d,bound", [(8, 2.0**-25), (16, 2.07e-8), (32, 2.09e-8), (64, 1.85e-8), (128, 1.72e-8),
                                     (400, 1.70e-8)])
def test_score_error_against_float64(d, bound):
    """Root mean square error of the scores relative to |a| |b|.  From d = 16 on
    the bound is what float32 operands as three exact bfloat16 pieces and six
    products reach on the same rows, where the rounding of the sums counts; at
    d = 8 the two planes' own 2^-24 an operand does (half of 2^-24 in all)."""
    C, U, m = 500, 500, 1000
    pb = make_problem("identity", "dot", "ranking", n=3000, m=m, d=d, C=C, U=U, S=2, sigma=1.0, zipf=0.2, seed=1)
    gm = GpuModel(pb)
    try:
        got, _ = gpu_inspect(gm, 0, m, 0)
    finally:
        gm.close()
    om = oracle_model(pb)
    want = O.inspect_step(om, 0, 0, pb.src, None, pb.dst, C, U, pb.seed, 0)
    negs = O.step_negatives(om, 0, 0, O.make_chunks(m, C, None, "consecutive"), pb.seed, U)
    norm = np.linalg.norm(om.emb[0], axis=1)
    sq = []
    for c, (a, b) in enumerate(zip(got, want)):
        q, t = norm[pb.src[C * c:C * (c + 1)]], norm[np.r_[pb.dst[C * c:C * (c + 1)], negs[c][0]]]
        e = (a["S0"] - b["S0"]) / (q[:, None] * t)
        sq.append(e[~np.eye(C, C + U, dtype=bool)] ** 2)   # a chunk's own destination is no candidate
    assert np.sqrt(np.mean(np.concatenate(sq))) <= bound
