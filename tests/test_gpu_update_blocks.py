"""The sorted update on both sides of the numbers of positions at which its
blocks grow from 8 to 32 (16,384 with fewer than 1,024 rows a table; else
32,768, uniform draws counted half), and well past them: one step against the
oracle."""
import numpy as np
import pytest

from oracle import pbg_oracle as O
from tests.pbg_cases import GpuModel, make_problem, oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [8, 32])
@pytest.mark.parametrize("n,U,d", [(1500, 511, 16), (1500, 512, 16), (1500, 513, 16), (40, 512, 130), (40, 513, 130),
                                   (300, 512, 260), (300, 513, 260)])
def test_update_around_the_block_line(n, U, d, S):
    """Chunks of 512 edges: 16,368, 16,384 and 16,400 positions, and four times
    as many."""
    _check(n, U, d, S)


@pytest.mark.parametrize("n,U,d", [(1023, 536, 16), (1024, 536, 16), (1500, 537, 130), (3000, 536, 260), (3000, 537, 260)])
def test_update_around_the_line_of_large_tables(n, U, d):
    """21 chunks of 512 edges: 32,760 and 32,781 of 44,016 and 44,058 positions."""
    _check(n, U, d, 21)


def _check(n, U, d, S):
    """A row sums up to 20,000 float32 terms (the Zipf head among 40 rows): 20,000 x 2^-24 =
    1.2e-3 of its absolute sum at worst."""
    pb = make_problem("translation", "dot", "logistic", n=n, m=S * 512, d=d, C=512, U=U, S=S, seed=3)
    gm = GpuModel(pb)
    try:
        gl = gm.train()
        st = gm.state()
    finally:
        gm.close()
    om = oracle_model(pb)
    ol = O.train_bucket(om, pb.i, pb.j, pb.src, pb.rel_ids, pb.dst, pb.C, pb.U, pb.S, pb.lr, pb.seed)
    assert abs(gl - ol) <= 1e-5 * max(1.0, abs(ol))
    for got, want in ((st["G"][0], om.G[0]), (st["emb"][0], om.emb[0])):
        assert np.max(np.abs(got - want)) <= 1.2e-3 * max(1.0, float(np.max(np.abs(want))))
