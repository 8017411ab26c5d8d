"""fp32 products as products of two fp16 pieces (contractions of 256 and more per workgroup): every tile and operand order,
edges, and the scales of rows that a sample does not tell the truth about.  Which kernel a shape gets is checked on the host
(test_fp32_plan.py).

Error bound of a sum on ordinary data: an operand is off by 2^-23 of itself (its two pieces); the product that is left out is
below 2^-22 |a b|; every matrix instruction adds 32 products with an error of at most one unit in the last place of a sum that
never exceeds sum |a b|, three of them per 32 k; up to 64 K ranges are added:
|got - exact| <= (2^-23 (3 ceil(K / 32) + 64) + 2^-21) sum |a b| + 2^-144,
the last term because a result and the partial sums of up to 64 K ranges are whole multiples of 2^-149.  Whatever the data, the
bound of products of three bf16 pieces holds (_strict)."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
BIG = torch.finfo(torch.float32).max


@pytest.fixture(scope="module")
def grass():
    import paper_2505_18976_amd as g
    g.load_library()
    return g


def _dev():
    return torch.device("cuda:0")


def _bound(A, B):
    return (2.0 ** -23 * (3 * -(-A.shape[1] // 32) + 64) + 2.0 ** -21) * (A.double().abs() @ B.double().abs().T.contiguous()) + 2.0 ** -144


def _strict_bound(A, B):
    """2^-23 (6 ceil(K / 16) + 65) sum |a b|, and 2^-144 as above: nothing for values that are small beside others of their row."""
    return (6 * -(-A.shape[1] // 16) + 65) * 2.0 ** -23 * (A.double().abs() @ B.double().abs().T.contiguous()) + 2.0 ** -144


def _check(got, A, B, bound=_bound):
    """got = A B^T within the bound, where that is an fp32 number."""
    ref = A.double() @ B.double().T.contiguous()
    off = ((got.double() - ref).abs() > bound(A, B)) & (ref.abs() <= BIG)
    assert not bool(off.any()), (int(off.sum()), off.nonzero()[:5].tolist())
    return ref


def _strict(got, A, B):
    return _check(got, A, B, _strict_bound)


# Shapes (rows of the first operand, of the second, K) and the kernel that they get with and without a workspace: tile of a
# product of two fp16 pieces, "-" one of three bf16 pieces, "head+tail" a cut one.
SCORES = {
    (2_048, 8_192, 257): ("256", "256"), (2_048, 8_192, 512): ("256", "256"), (2_040, 8_190, 600): ("256", "256"),
    (2_048, 8_192, 1_000): ("256", "256"), (130, 70_001, 700): ("256+-", "256+128"),
    (130, 130, 4_100): ("-", "128"), (1, 1, 257): ("-", "128"), (129, 1_000, 1_023): ("-", "128"), (1_000, 4_000, 1_000): ("128", "128"),
    (501, 39_999, 256): ("128", "128"), (60, 200, 5_000): ("-", "128"), (40, 300, 700): ("-", "128"),
    (100, 70_001, 600): ("128", "128"), (300, 50_000, 270): ("128", "128"), (70, 90, 20_001): ("128", "128"), (40, 5_000, 515): ("-", "128"),
    (128, 65_536, 512): ("128x256", "128x256"), (128, 33_000, 1_000): ("128x256", "128x256"), (5, 33_000, 2_048): ("128", "128x256"),
    (1, 40_000, 1_100): ("-", "128x256"),
}
# K-major both: rows and columns of G
FIMS = {(5_000, 1_024): "128", (2_000, 1_030): "128", (501, 3_999): "256", (500, 4_000): "256", (257, 4_002): "256", (300, 4_000): "256"}
# test rows, train rows, columns: kernels of the two products of a Selective-Mask step; up to 128 test rows the backward one has the
# gradient in its registers, on tiles of 64 x 128 for up to 64 rows and of 128 x 256 above
STEPS = {
    (100, 1_000, 100_001): ("128x256", "grad"), (65, 1_000, 131_073): ("128x256", "grad"), (128, 1_000, 90_001): ("128x256", "grad"),
    (100, 300, 257): ("-", "grad"), (128, 300, 1_027): ("-", "grad"), (17, 259, 4_098): ("-", "grad"), (64, 300, 129): ("-", "grad"),
    (65, 300, 127): ("-", "grad"), (33, 1_000, 128): ("-", "grad"), (1, 1_000, 255): ("-", "grad"), (128, 600, 33_000): ("128", "grad"),
    (256, 1_000, 65_536): ("256", "256"), (129, 1_000, 4_099): ("-", "128"),
}


@pytest.mark.parametrize("M,N,K", [(2_048, 8_192, 256), (2_040, 8_190, 300), (100, 70_001, 288), (128, 65_536, 260), (33, 100_000, 300),
                                   (64, 40_001, 511), (5, 33_000, 256)] + [q for q in SCORES if q[2] < 4_100])
@pytest.mark.parametrize("pad", [0, 1])
def test_row_major(grass, M, N, K, pad):
    te = synth.dense_normal(M, K + pad, seed=1, device=_dev())[:, :K]
    tr = synth.dense_normal(N, K + 3 * pad, seed=2, device=_dev())[:, :K]
    for ws in ({}, {"ws": None}):
        got = grass.grass_score(tr, te, **ws)
        ref = _check(got, te, tr)
        if K <= 300:                         # seen 2.1e-7; the products of pieces left out at most 4e-8, one more lost 1e-4
            assert float((got.double() - ref).norm() / ref.norm()) <= 3e-7


@pytest.mark.parametrize("N,k", [(300, 4_000), (290, 4_001), (257, 4_002), (300, 4_003), (300, 130), (300, 131), (300, 257),
                                 (300, 1), (300, 2), (299, 3), (300, 4), (300, 5), (4_000, 190), (70_001, 67),
                                 (5_000, 1_024), (2_000, 1_030), (501, 3_999)])
def test_both_operands_k_major(grass, N, k):
    G = synth.dense_normal(N, k, seed=3, device=_dev())
    F = grass.grass_fim(G)
    assert torch.equal(F, F.T)
    _check(F * N, G.T, G.T)                  # the scaling by 1 / N and back adds two roundings, inside the bound's 64


@pytest.mark.parametrize("m,n,p", [(3, 300, 1), (2, 257, 3), (3, 300, 5), (3, 300, 4_099), (256, 300, 65_536), (255, 299, 65_533),
                                   (100, 290, 70_002), (128, 600, 33_000), (256, 1_000, 65_536), (129, 1_000, 4_099)])
def test_second_operand_k_major(grass, m, n, p):
    """The backward product of a Selective-Mask step: its gradient is compared with that of double precision.  Masked scores,
    their correlation and the row c behind them keep 1e-5 of the largest entry."""
    G, Gt = synth.dense_normal(n, p, seed=7, device=_dev()), synth.dense_normal(m, p, seed=8, device=_dev())
    S = synth.dense_normal(1, p, seed=9, device=_dev(), std=0.5).reshape(-1).contiguous()
    A = synth.dense_normal(m, n, seed=10, device=_dev())
    grad, _ = grass.grass_selective_mask_grad(G, Gt, A, S, 1e-3, 1.0)
    sig, g, gt, a = torch.sigmoid(S.double()), G.double(), Gt.double(), A.double()
    b = (gt * sig ** 2) @ g.T.contiguous()
    da, db = a - a.mean(1, keepdim=True), b - b.mean(1, keepdim=True)
    na, nb = da.norm(dim=1, keepdim=True), db.norm(dim=1, keepdim=True)
    c = (da / (na * nb) - (da * db).sum(1, keepdim=True) / (na * nb ** 3) * db) / m
    ds = sig * (1 - sig)
    ref = 2 * sig * ds * (gt * (c @ g)).sum(0) - 1e-3 * ds
    assert float((grad.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("m,n,p", [(1, 256, 255), (100, 300, 257), (128, 300, 1_027), (17, 259, 4_098), (64, 300, 129),
                                   (65, 300, 127), (33, 1_000, 128), (1, 1_000, 255)])
@pytest.mark.parametrize("spoil", ["zeros", "late", "far", "infinite"])
def test_gradient_of_columns_that_the_sample_misjudges(grass, m, n, p, spoil):
    """The gradient out of the backward product's registers, with columns of G that send their tile through the second attempt."""
    G, Gt = synth.dense_normal(n, p, seed=7, device=_dev()), synth.dense_normal(m, p, seed=8, device=_dev())
    S = synth.dense_normal(1, p, seed=9, device=_dev(), std=0.5).reshape(-1).contiguous()
    A = synth.dense_normal(m, n, seed=10, device=_dev())
    if spoil == "zeros":                     # nothing in the sample, small behind it
        G[:200, 5], G[200:, 5] = 0.0, G[200:, 5] * 2.0 ** -20
        G[:, p - 1] = 0.0
    else:                                    # too large for the sample, of wide range; test gradients are zero there
        G[100, 7] = {"late": 2.0 ** 12, "far": 2.0 ** 30, "infinite": float("inf")}[spoil]
        Gt[:, 7] = 0.0
    sig, g, gt, a = torch.sigmoid(S.double()), G.double(), Gt.double(), A.double()
    g0 = g.nan_to_num(0.0, 0.0, 0.0)
    b = (gt * sig ** 2) @ g0.T.contiguous()
    da, db = a - a.mean(1, keepdim=True), b - b.mean(1, keepdim=True)
    na, nb = da.norm(dim=1, keepdim=True), db.norm(dim=1, keepdim=True)
    c = (da / (na * nb) - (da * db).sum(1, keepdim=True) / (na * nb ** 3) * db) / m
    ds = sig * (1 - sig)
    ref = 2 * sig * ds * (gt * (c @ g0)).sum(0) - 1e-3 * ds
    grad, _ = grass.grass_selective_mask_grad(G, Gt, A, S, 1e-3, 1.0)
    if spoil == "infinite":                  # 0 times infinity in every masked score of train row 100
        assert bool(torch.isnan(grad).all())
        return
    assert float((grad.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


def test_gradient_of_more_train_rows_than_32_bit_offsets_reach(grass):
    """2^26 train rows: the rows of the backward product's first operand are too far apart for the kernel that has the gradient
    in its registers.  All train rows but 400 are zero, so the error bound of a sum is that of 400 terms."""
    n, m, p, rows = 1 << 26, 2, 4, 400
    G, A = torch.zeros(n, p, device=_dev()), torch.zeros(m, n, device=_dev())
    at = torch.arange(rows, device=_dev()) * 167_771
    G[at], A[:, at] = synth.dense_normal(rows, p, seed=7, device=_dev()), synth.dense_normal(m, rows, seed=10, device=_dev())
    Gt, S = synth.dense_normal(m, p, seed=8, device=_dev()), synth.dense_normal(1, p, seed=9, device=_dev()).reshape(-1)
    grad, _ = grass.grass_selective_mask_grad(G, Gt, A, S.contiguous(), 1e-3, 1.0)
    sig, g, gt, a = torch.sigmoid(S.double()), G[at].double(), Gt.double(), A[:, at].double()
    b = (gt * sig ** 2) @ g.T.contiguous()
    ma, mb = a.sum(1, keepdim=True) / n, b.sum(1, keepdim=True) / n
    na, nb = ((a ** 2).sum(1, keepdim=True) - n * ma ** 2).sqrt(), ((b ** 2).sum(1, keepdim=True) - n * mb ** 2).sqrt()
    corr = ((a * b).sum(1, keepdim=True) - n * ma * mb) / (na * nb)
    c = ((a - ma) / (na * nb) - corr / nb ** 2 * (b - mb)) / m
    ds = sig * (1 - sig)
    ref = 2 * sig * ds * (gt * (c @ g)).sum(0) - 1e-3 * ds
    assert float((grad.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("m,n,p", [(100, 1_000, 20_001), (65, 600, 33_000), (128, 513, 8_193), (66, 300, 5_003),
                                   (100, 1_000, 100_001), (65, 1_000, 131_073), (128, 1_000, 90_001)])
@pytest.mark.parametrize("std", [0.5, 15.0, "trained"])
@pytest.mark.parametrize("spoil", [False, True])
def test_weights_applied_on_the_way_in(grass, m, n, p, std, spoil):
    """The forward product weighs the test gradients as it reads them: ragged p, weights from 1 to nothing, rows that the sample
    misjudges.  Objective and gradient against double precision."""
    G, Gt = synth.dense_normal(n, p, seed=7, device=_dev()), synth.dense_normal(m, p, seed=8, device=_dev())
    S = synth.dense_normal(1, p, seed=9, device=_dev(), std=0.5 if std == "trained" else std).reshape(-1).contiguous()
    if std == "trained":                     # one column in 100 is kept, the others next to nothing: samples miss the weights of one
        S = torch.where(torch.arange(p, device=_dev()) % 100 == 57, S + 2.0, S - 12.0)
    if spoil:
        Gt[3, 50], Gt[4, p - 1], Gt[5] = 2.0 ** 12, 2.0 ** 14, Gt[5] * 2.0 ** -60
        Gt[6, : p // 2], S[p // 2:] = 0.0, S[p // 2:] - 12.0
    sig, g, gt = torch.sigmoid(S.double()), G.double(), Gt.double()
    A = (gt @ g.T.contiguous()).float()
    b, a = (gt * sig ** 2) @ g.T.contiguous(), A.double()
    da, db = a - a.mean(1, keepdim=True), b - b.mean(1, keepdim=True)
    na, nb = da.norm(dim=1, keepdim=True), db.norm(dim=1, keepdim=True)
    corr = (da * db).sum(1, keepdim=True) / (na * nb)
    c = (da / (na * nb) - corr / nb ** 2 * db) / m
    ds = sig * (1 - sig)
    ref = 2 * sig * ds * (gt * (c @ g)).sum(0) - 1e-6 * ds
    grad, obj = grass.grass_selective_mask_grad(G, Gt, A, S, 1e-6, 1.0)
    assert abs(float(obj) - float(corr.mean() - 1e-6 * sig.sum())) <= 1e-5
    assert float((grad.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


def _odd_rows(X):
    """Rows that a sample of the first 32 k (and of three more groups in long ranges) misjudges."""
    K = X.shape[1]
    X[0] *= 2.0 ** -120
    X[1] *= 2.0 ** 40
    X[2] = 0.0
    X[3, :K - 3] = 0.0                       # nothing but the last three, of ordinary size
    X[4, :100] = 0.0
    X[4, 100:] *= 2.0 ** -40                 # zero in the sample and far below the rest of the tile
    X[5, 40] = 2.0 ** 7                      # above the sample: fits
    X[6, 41] = 2.0 ** 12                     # does not
    X[7, 42] = 2.0 ** 22                     # wide range
    X[8, 43] = BIG
    X[9, 200:] *= 2.0 ** -20
    X[10, 3] = 2.0 ** 25                     # in the sample
    X[11] = 2.0 ** -149 * torch.randint(-5, 6, (K,), device=X.device)
    return X


@pytest.mark.parametrize("M,N,K", [(40, 300, 257), (300, 40, 512), (20, 40_000, 300), (130, 70_001, 260), (2_048, 8_192, 256),
                                   (60, 200, 5_000), (40, 300, 700), (1_000, 4_000, 1_000), (128, 33_000, 1_000), (2_048, 8_192, 512)])
def test_rows_that_the_sample_misjudges(grass, M, N, K):
    te = _odd_rows(synth.dense_normal(M, K, seed=11, device=_dev()))
    tr = _odd_rows(synth.dense_normal(N, K, seed=12, device=_dev()))
    for a, b in ((te, synth.dense_normal(N, K, seed=13, device=_dev())), (synth.dense_normal(M, K, seed=14, device=_dev()), tr)):
        for ws in ({}, {"ws": None}):
            _strict(grass.grass_score(b, a, **ws), a, b)


@pytest.mark.parametrize("spike", [2.0 ** 13, 2.0 ** 22, 2.0 ** 40, BIG])
@pytest.mark.parametrize("M,N,K", [(40, 300, 300), (300, 5_000, 256), (60, 200, 5_000), (1_000, 4_000, 1_000), (128, 33_000, 1_000),
                                   (2_048, 8_192, 1_000)])
def test_large_values_that_meet_zeros(grass, spike, M, N, K):
    """A row with one huge value where the other operand is zero, in the sample and outside: the sums are those of the rest, to
    the bits of the rest."""
    te, tr = synth.dense_normal(M, K, seed=15, device=_dev()), synth.dense_normal(N, K, seed=16, device=_dev())
    tr[:, 5] = tr[:, 100] = 0.0
    te[1, 5], te[17, 100] = spike, -spike
    for ws in ({}, {"ws": None}):
        _strict(grass.grass_score(tr, te, **ws), te, tr)
    _strict(grass.grass_score(te, tr), tr, te)


@pytest.mark.parametrize("N,k", [(300, 130), (400, 1_003), (5_000, 1_024), (500, 4_000)])
def test_large_values_that_meet_zeros_k_major(grass, N, k):
    G = synth.dense_normal(N, k, seed=17, device=_dev())
    G[5] = G[100] = 0.0
    G[5, 3], G[100, 77] = BIG / 4, 2.0 ** 30
    ref = G.T.double() @ G.double()
    got = grass.grass_fim(G).double() * N
    ok = ref.abs() <= BIG
    assert bool(((got - ref).abs() <= _strict_bound(G.T, G.T))[ok].all()) and bool(torch.isinf(got[~ok]).all())


@pytest.mark.parametrize("M,N,K", [(60, 200, 5_000), (1_000, 4_000, 1_000),           # 128 x 128 (the first without a workspace)
                                   (128, 33_000, 1_000), (2_048, 8_192, 1_000)])      # 128 x 256, 256 x 256
@pytest.mark.parametrize("spike", [2.0 ** 13, 2.0 ** 22, 2.0 ** 30])
@pytest.mark.parametrize("at", [5, 700])
def test_sums_that_miss_the_large_value_of_their_row(grass, M, N, K, spike, at):
    """A test row has one large value; 0 to 12 of every 16 train rows are zero there, the others are not.  Their sums are those of
    the rest of the row, to the bits of the rest, whatever the neighbouring sums are."""
    te, tr = synth.dense_normal(M, K, seed=41, device=_dev()), synth.dense_normal(N, K, seed=42, device=_dev())
    te[[3, 17, M - 1], at] = spike
    block, inside = torch.arange(N, device=_dev()) // 16, torch.arange(N, device=_dev()) % 16
    zero = inside < torch.tensor([0, 1, 4, 7, 8, 12], device=_dev())[block % 6]
    tr[zero, at] = 0.0
    for ws in ({}, {"ws": None}):
        _strict(grass.grass_score(tr, te, **ws), te, tr)
    if N <= 4_000:
        _strict(grass.grass_score(te, tr), tr, te)


@pytest.mark.parametrize("M,N,K", [(60, 200, 5_000), (1_000, 4_000, 1_000), (128, 33_000, 1_000), (2_048, 8_192, 1_000)])
@pytest.mark.parametrize("fall", [12, 20, 24, 27])
def test_rows_whose_first_values_tower_above_the_rest(grass, M, N, K, fall):
    te, tr = synth.dense_normal(M, K, seed=43, device=_dev()), synth.dense_normal(N, K, seed=44, device=_dev())
    te[:40, 20:] *= 2.0 ** -fall
    tr[1::3, :20] = 0.0
    tr[5::48, :K - 40] = 0.0                 # and rows with few values
    for ws in ({}, {"ws": None}):
        _strict(grass.grass_score(tr, te, **ws), te, tr)


@pytest.mark.parametrize("N,k", [(5_000, 1_024), (500, 4_000), (501, 3_999)])         # 128 x 128, 256 x 256, both K-major
@pytest.mark.parametrize("spike", [2.0 ** 13, 2.0 ** 22, 2.0 ** 30])
def test_columns_that_miss_the_large_value_of_another(grass, N, k, spike):
    G = synth.dense_normal(N, k, seed=45, device=_dev())
    col = torch.arange(k, device=_dev())
    for row in (3, N - 1):
        G[row, col % 16 < (col // 16) % 13] = 0.0
        G[row, 40 + row % 16] = spike
    G[20:, 100] *= 2.0 ** -20                # the first values tower above the rest,
    G[:20, col % 48 == 7] = 0.0              # where others are zero
    _strict(grass.grass_fim(G) * N, G.T, G.T)


@pytest.mark.parametrize("N,k", [(3_000, 1_100), (1_000, 1_100), (300, 1_024), (4_096, 2_080), (5_000, 4_096)])
@pytest.mark.parametrize("peak", [2.0 ** 4, 2.0 ** 12, 2.0 ** 24])
def test_rows_times_a_nearly_diagonal_matrix(grass, N, k, peak):
    """Preconditioning with the inverse of a matrix: the diagonal towers above the rest of its rows, also where it lies in the last
    group of a ragged k, and some rows are zero there."""
    G, W = synth.dense_normal(N, k, seed=48, device=_dev()), synth.dense_normal(k, k, seed=49, device=_dev())
    W = W + W.T
    W.diagonal().mul_(peak)
    W[k // 2, k // 2] = 0.0
    G[::3, ::2] = 0.0
    got = grass.grass_ifvp(G, W)
    _strict(got, G, W)
    assert float((got - G @ W).norm()) <= 4e-6 * float(got.norm())


def test_rows_with_one_value(grass):
    """The sums are single products of values that are small beside the largest of their row."""
    te, tr = synth.dense_normal(300, 1_000, seed=46, device=_dev()), torch.zeros(5_000, 1_000, device=_dev())
    tr[torch.arange(5_000), torch.arange(5_000) % 1_000] = synth.dense_normal(1, 5_000, seed=47, device=_dev())[0]
    for ws in ({}, {"ws": None}):
        _strict(grass.grass_score(tr, te, **ws), te, tr)
        _strict(grass.grass_score(te, tr, **ws), tr, te)


@pytest.mark.parametrize("M,N,K", [(70, 90, 20_001), (40, 5_000, 515), (300, 50_000, 270), (2_048, 8_192, 257)])
def test_non_finite_operands(grass, M, N, K):
    te, tr = synth.dense_normal(M, K, seed=31, device=_dev()), synth.dense_normal(N, K, seed=32, device=_dev())
    for x in (te, tr):
        x[3, 5], x[4, K - 1], x[7, 9] = float("inf"), float("nan"), float("-inf")
        x[8, 1], x[8, K - 1] = float("inf"), float("-inf")
        x[9, 40] = 2.0 ** 30                 # next to infinities, a scale that has to be found again
    ref = te.double() @ tr.double().T.contiguous()
    for ws in ({}, {"ws": None}):
        got = grass.grass_score(tr, te, **ws).double()
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
        assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
        ok = torch.isfinite(ref)
        te0, tr0 = te.nan_to_num(0.0, 0.0, 0.0), tr.nan_to_num(0.0, 0.0, 0.0)
        assert bool(((got - ref).abs() <= _strict_bound(te0, tr0))[ok].all())


@pytest.mark.parametrize("p,chunk", [(1_300, 512), (9_000, 4_096)])       # three bf16 pieces; two fp16 ones in 8 K ranges
@pytest.mark.parametrize("spoilt", [1, 4])
def test_accumulated_chunks(grass, p, chunk, spoilt):
    """Gaussian projection in column chunks that are added up, the last one short; infinities and a late large value: in one row a
    few sums are computed again, in four the tile."""
    k = 40
    g = synth.dense_normal(20, p, seed=34, device=_dev())
    last = p // chunk * chunk
    for i, at in ((8, 200), (8, chunk + 188), (3, 5), (3, last + 3), (4, chunk + 88), (7, last - 60))[:2 if spoilt == 1 else 6]:
        g[i, at] = {3: float("inf"), 4: float("nan"), 7: float("-inf"), 8: 2.0 ** 20}[i]
    P = grass.grass_gauss_matrix(0, 9, p, k, 0, p, device=_dev())
    got = grass.grass_gauss_project(g, k, 0, 9, chunk, 0).double()
    ref = g.double() @ P.double().T.contiguous()
    assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
    ok = torch.isfinite(ref)
    assert bool(((got - ref).abs() <= _strict_bound(g.nan_to_num(0.0, 0.0, 0.0), P))[ok].all())


def test_gradients_of_a_relu_network_take_the_time_of_dense_ones(grass):
    """Scores and a Selective-Mask step on gradients with runs of zeros (dead neurons), columns of zeros (200 of 784 inputs) and row
    norms over 2^8, against dense ones: rows and columns of which a sample shows nothing stay where the others are.  Seen 0.97 to
    1.03 times the dense time; 2.0 to 2.9 where one such row sends its tile elsewhere."""
    n, m, p = 1_000, 100, synth.mlp_num_params()
    gen = torch.Generator(device=_dev()).manual_seed(21)
    G, Gt = synth.dense_normal(n, p, seed=22, device=_dev(), std=0.1), synth.dense_normal(m, p, seed=23, device=_dev(), std=0.1)
    S = synth.dense_normal(1, p, seed=24, device=_dev(), std=0.1).reshape(-1).contiguous()
    A = grass.grass_score(G, Gt)

    def times():
        out = []
        for f in (lambda: grass.grass_score(G, Gt), lambda: grass.grass_selective_mask_grad(G, Gt, A, S, 1e-6, 1.0)):
            f()
            runs = []
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                f()
                b.record()
                b.synchronize()
                runs.append(a.elapsed_time(b))
            out.append(sorted(runs)[2])
        return out

    dense = times()
    off = torch.randperm(784, generator=torch.Generator().manual_seed(1))[:200].to(_dev())
    for X, rows, seed in ((G, n, 25), (Gt, m, 26)):
        X.copy_(synth.mlp_relu_gradients(rows, seed=seed, device=_dev()))
        X[:, :784 * 1_024].unflatten(1, (1_024, 784))[:, :, off] = 0
        X.mul_(torch.exp2(8 * torch.rand(rows, 1, device=_dev(), generator=gen)))
    relu = times()
    assert relu[0] <= 1.3 * dense[0] and relu[1] <= 1.3 * dense[1], (dense, relu)
    got, ref = grass.grass_score(G[:200], Gt).double(), Gt.double() @ G[:200].double().T.contiguous()
    assert float((got - ref).norm(dim=0).div(ref.norm(dim=0)).max()) <= 2e-5
