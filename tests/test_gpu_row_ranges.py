"""Gradients whose factors span many binades: candidates that only small
probabilities reach, and rows of very unlike size in one chunk.  A row's first
Adagrad step is lr g / |g|, so every row's gradient counts relative to its own
size."""
import numpy as np
import pytest

from oracle import pbg_oracle as O
from paper_1903_12287_amd import synth
from tests.pbg_cases import GpuModel, make_problem, oracle_model, teacher_forced_step

pytestmark = pytest.mark.gpu

HOT, COLD, GIANT = 100, 300, 6


def _problem(loss, C, U, m, d, giant, gap, seed=3, op="identity"):
    """Edges join hot rows (about 2 along axis 0).  Cold rows, reached by the
    uniform draws only, lie opposite to them: their scores are below the hot
    ones by `gap`'s range.  Giant rows (2^giant, or none) lie opposite to them
    too: no probability is left for them, and no hinge selects them."""
    pb = make_problem(op, "dot", loss, R=1, n=HOT + COLD + GIANT, m=m, d=d, C=C, U=U, S=4, seed=seed)
    rng = synth.rng_for(seed)
    x = 0.3 * rng.standard_normal((pb.n, d))
    x[:HOT, 0] = 2.0
    x[HOT:, 0] = -np.linspace(*gap, COLD + GIANT) / 2.0 + 2.0
    if giant is not None:
        x[HOT + COLD:] = 0.0
        x[HOT + COLD:, 0] = -(2.0**giant)
    pb.parts[0][...] = x.astype(np.float32)
    if pb.rel is not None:
        pb.rel[...] = 1.0
    pb.src, pb.dst = (rng.integers(0, HOT, m) for _ in range(2))
    return pb


def _check(pb, eps):
    gm = GpuModel(pb)
    try:
        _, gl, ol, worst = teacher_forced_step(gm, 0, len(pb.src), 0, eps)
    finally:
        gm.close()
    assert abs(gl - ol) <= 1e-5 * max(1.0, abs(ol))
    assert worst <= 1.0


# (C, U, edges, d): both column widths and a remainder of every tile
SHAPES = [(100, 150, 230, 33), (300, 260, 560, 100), (70, 130, 70, 250), (64, 64, 64, 16)]


@pytest.mark.parametrize("C,U,m,d", SHAPES)
@pytest.mark.parametrize("giant", [None, 20, 45])
@pytest.mark.parametrize("loss", ["logistic", "softmax"])
def test_small_probabilities(loss, giant, C, U, m, d):
    """Scores down to -40 (probabilities of 2^-60; |g| down to Adagrad's
    epsilon of 1e-10).  A score's error is about d 2^-24 of its absolute sum of
    up to 100, which is the relative error of its probability: 1e-4 bounds it
    with the gradient's own 1e-5."""
    _check(_problem(loss, C, U, m, d, giant, (10.0, 44.0)), 1e-4)


@pytest.mark.parametrize("C,U,m,d", SHAPES + [(130, 300, 400, 113), (20, 40, 50, 8)])
@pytest.mark.parametrize("giant", [None, 20, 45, 90])
@pytest.mark.parametrize("op", ["identity", "diagonal"])
def test_ranking_rows_of_unlike_size(op, giant, C, U, m, d):
    """Candidates up to 2^90 that no hinge selects beside ordinary ones, rows of
    2^-33 that select candidates no other query does, and rows of zeros."""
    pb = _problem("ranking", C, U, m, d, giant, (-1.0, 30.0), op=op)
    pb.parts[0][:10] *= np.float32(2.0**-33)
    pb.parts[0][HOT:HOT + 10] = 0.0
    pb.src[::7] = np.arange(len(pb.src[::7])) % 10
    pb.dst[3::11] = np.arange(len(pb.dst[3::11])) % 10
    _check(pb, 1e-5)


@pytest.mark.parametrize("loss", ["ranking", "logistic", "softmax"])
def test_scores_near_the_largest_float(loss):
    """A candidate of 2^118 that every hinge selects: its scores, 2^119, are
    finite, and so are the loss and the embeddings (its accumulators are not)."""
    pb = _problem(loss, 100, 150, 230, 33, None, (10.0, 20.0))
    pb.parts[0][HOT + COLD:] = 0.0
    pb.parts[0][HOT + COLD:, 0] = 2.0**118
    gm = GpuModel(pb)
    try:
        gl = gm.train()
        emb = gm.state()["emb"][0]
    finally:
        gm.close()
    with np.errstate(all="ignore"):
        ol = O.train_bucket(oracle_model(pb), 0, 0, pb.src, None, pb.dst, pb.C, pb.U, pb.S, pb.lr, pb.seed)
    assert abs(gl - ol) <= 1e-5 * abs(ol)
    assert np.isfinite(emb).all()


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 3e38])
@pytest.mark.parametrize("op,cmp", [("identity", "dot"), ("translation", "cos")])
@pytest.mark.parametrize("loss", ["ranking", "logistic", "softmax"])
def test_a_row_that_is_no_number_stays_in_its_chunk(loss, op, cmp, value):
    """Whatever such a row does to its own chunk's products, rows that only the
    step's other chunks touch get the bits that they get without it."""
    C, U, m = 100, 28, 300
    pb = make_problem(op, cmp, loss, R=1, n=900, m=m, d=33, C=C, U=U, S=3, seed=5, zipf=0.5)
    bad = 0
    pb.src[pb.src == bad] = 1
    pb.dst[pb.dst == bad] = 1
    pb.src[3] = pb.dst[20] = bad   # chunk 0
    negs = O.step_negatives(oracle_model(pb), 0, 0, O.make_chunks(m, C, None, "consecutive"), pb.seed, U)
    assert not any((n == bad).any() for pair in negs[1:] for n in pair)
    first = np.r_[pb.src[:C], pb.dst[:C], negs[0][0], negs[0][1]]
    others = np.setdiff1d(np.r_[pb.src[C:], pb.dst[C:], negs[1][0], negs[1][1], negs[2][0], negs[2][1]], first)
    assert len(others) > 100
    got = []
    for row in (pb.parts[0][bad].copy(), np.float32(value)):
        pb.parts[0][bad] = row
        gm = GpuModel(pb)
        try:
            gm.train()
            got.append(gm.state())
        finally:
            gm.close()
    for key in ("emb", "G"):
        a, b = (g[key][0][others] for g in got)
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(a, b)
