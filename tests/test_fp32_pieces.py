"""Every one of the six products of bf16 pieces that make up an fp32 product, in every tile and operand order.

Leaving one of them out changes a product of normal data by at least 2.4e-6 in the 2-norm (the CPU test below); the sums
over up to 200 terms here are good to 2.1e-7 at most.  Bar in between: 8e-7."""
import numpy as np
import pytest
import torch

import synth

BAR = 8e-7


def _pieces(x):
    out = []
    for _ in range(3):
        u = x.view(np.uint32).astype(np.uint64)
        h = ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)
        out.append(h.astype(np.float64))
        x = x - h
    assert not x.any()
    return out


def test_bar_sees_a_lost_product():
    rng = np.random.default_rng(0)
    a, b = (rng.standard_normal((200, 200)).astype(np.float32) for _ in range(2))
    A, B, ref = _pieces(a), _pieces(b), a.astype(np.float64) @ b.T.astype(np.float64)
    kept = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]
    off = lambda pairs: np.linalg.norm(sum(A[i] @ B[j].T for i, j in pairs) - ref) / np.linalg.norm(ref)
    assert off(kept) < 1e-8
    assert all(off([q for q in kept if q != p]) > 2.4e-6 for p in kept)


def _dev():
    return torch.device("cuda:0")


def _off(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(130, 130, 200),          # 128 x 128, three K ranges
                                   (2_048, 8_192, 200), (2_040, 8_190, 195),     # 256 x 256
                                   (33, 100_000, 200), (33, 99_999, 197)])       # 64 x 512
def test_row_major(M, N, K):
    import paper_2505_18976_amd as grass
    te, tr = synth.dense_normal(M, K, seed=1, device=_dev()), synth.dense_normal(N, K, seed=2, device=_dev())
    ref = te.double() @ tr.double().T.contiguous()
    for ws in ({}, {"ws": None}):
        assert _off(grass.grass_score(tr, te, **ws), ref) <= BAR


@pytest.mark.gpu
@pytest.mark.parametrize("N,k", [(200, 130), (199, 131), (100, 4_000), (99, 4_001)])     # 128 x 128, 256 x 256
def test_both_operands_k_major(N, k):
    import paper_2505_18976_amd as grass
    G = synth.dense_normal(N, k, seed=3, device=_dev())
    assert _off(grass.grass_fim(G), G.T.double().contiguous() @ G.double() / N) <= BAR


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,p", [(3, 48, 4_096), (3, 47, 4_099), (256, 48, 65_536), (255, 47, 65_533)])
def test_second_operand_k_major(m, n, p):
    """The backward product R = C G of a Selective-Mask step.  Test gradients that are one where j mod m is the row and zero
    elsewhere make entry j of the gradient a quarter of R[j mod m][j] (logits 0: sigma = 1/2), and masked scores that are
    sums of p / m terms, so C is good to a few roundings."""
    import paper_2505_18976_amd as grass
    G = synth.dense_normal(n, p, seed=4, device=_dev())
    A = synth.dense_normal(m, n, seed=5, device=_dev())
    row = torch.arange(p, device=_dev()) % m
    Gt = torch.zeros(m, p, device=_dev())
    Gt[row, torch.arange(p, device=_dev())] = 1.0
    grad, _ = grass.grass_selective_mask_grad(G, Gt, A, torch.zeros(p, device=_dev()), 0.0, 1.0)
    a, g = A.double(), G.double()
    b = torch.zeros(m, n, dtype=torch.float64, device=_dev()).index_add_(0, row, g.T.contiguous()) / 4
    da, db = a - a.mean(1, keepdim=True), b - b.mean(1, keepdim=True)
    na, nb = da.norm(dim=1, keepdim=True), db.norm(dim=1, keepdim=True)
    C = (da / (na * nb) - (da * db).sum(1, keepdim=True) / (na * nb ** 3) * db) / m
    ref = (C[row] * g.T).sum(1) / 4
    assert _off(grad, ref) <= BAR
