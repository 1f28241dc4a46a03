"""One chunk whose score gradient dS passes 4 GiB (float32) and 2 GiB (bf16):
its last rows lie beyond what 32-bit byte offsets from the chunk's base reach."""
import numpy as np
import pytest
import torch

from oracle import pbg_oracle as O
from paper_1903_12287_amd import pbg
from tests.pbg_cases import GpuModel, make_problem, oracle_model

pytestmark = pytest.mark.gpu


def _reference(pb):
    """Loss, embeddings and accumulators after the step, float64 on the GPU in
    blocks of rows (identity operator, dot, logistic loss)."""
    dev = torch.device("cuda")
    step = O.make_chunks(len(pb.src), pb.C, None, "consecutive")
    (u_dst, u_src), = O.step_negatives(oracle_model(pb), 0, 0, step, pb.seed, pb.U)
    t = lambda a: torch.from_numpy(np.asarray(a, np.int64)).to(dev)
    src, dst = t(pb.src), t(pb.dst)
    E = torch.from_numpy(pb.parts[0]).to(dev).double()
    grad = torch.zeros_like(E)
    xs, xd = E[src], E[dst]
    p = (xs * xd).sum(1)
    loss = 2 * torch.nn.functional.softplus(-p).sum()
    dp = 2 * (torch.sigmoid(p) - 1)
    m, K = len(pb.src), len(pb.src) + pb.U - 1
    for q, qid, cid in ((xs, src, torch.cat([dst, t(u_dst)])), (xd, dst, torch.cat([src, t(u_src)]))):
        cand = E[cid]
        dn = torch.zeros_like(cand)
        for lo in range(0, m, 1024):
            qq = q[lo:lo + 1024]
            s = qq @ cand.T
            r = torch.arange(len(qq), device=dev)
            s[r, lo + r] = -torch.inf
            loss += torch.nn.functional.softplus(s).sum() / K
            ds = torch.sigmoid(s) / K
            grad.index_add_(0, qid[lo:lo + 1024], ds @ cand)
            dn += ds.T @ qq
        grad.index_add_(0, cid, dn)
    grad.index_add_(0, src, dp[:, None] * xd)
    grad.index_add_(0, dst, dp[:, None] * xs)
    G = (grad * grad).sum(1)
    emb = E - pb.lr * grad / (G.sqrt()[:, None] + O.EPS_ADAGRAD)
    emb = torch.where(G[:, None] > 0, emb, E)
    return float(loss), emb.cpu().numpy(), G.cpu().numpy()


@pytest.mark.parametrize("flags,tol", [(0, 1e-4), (pbg.F_BF16_SCORE, 2e-2)])
def test_chunk_of_more_than_4_gib(flags, tol):
    """16,384 edges against 81,920 candidates.  The accumulators' error is
    relative to the largest one; the embeddings' to the step size lr."""
    pb = make_problem("identity", "dot", "logistic", n=200_000, m=16_384, d=8, C=16_384, U=65_536, S=1, sigma=1.0,
                      zipf=0.3, seed=7)
    gm = GpuModel(pb, flags)
    try:
        loss = gm.train()
        st = gm.state()
    finally:
        gm.close()
    want_loss, emb, G = _reference(pb)
    assert abs(loss - want_loss) <= tol * abs(want_loss)
    assert np.linalg.norm(st["G"][0] - G) <= tol * np.linalg.norm(G)
    # the rows of the last edges, whose gradients are sums over the far rows of dS, and all of them
    for ids in (pb.src[-1000:], slice(None)):
        err = np.linalg.norm(st["emb"][0][ids] - emb[ids])
        assert err <= tol * np.linalg.norm(emb[ids] - pb.parts[0][ids])
