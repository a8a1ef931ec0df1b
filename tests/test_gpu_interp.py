"""GPU parity: tsne_kl_grad_fft (repulsion and Z by FFT-accelerated
interpolation) against the FP64 oracle of the same scheme
(oracle/interp.py) -- near-exact agreement, since both take the same grid,
boxes and weights -- and against the exact gradient within the scheme's
approximation error, which falls with the box side."""
import numpy as np
import pytest
import torch

import oracle
from helpers import random_graph_P, rel, say, sparse_to_dev, to_dev
from oracle import interp as I
from paper_2605_13928_amd import api, synth

pytestmark = pytest.mark.gpu

GRAD_RTOL = 1e-4  # FP32 output and FP32 attraction terms, as for tsne_kl_grad


def widen(S):
    return oracle.CSR(S.row_ptr, S.col, S.val.astype(np.float32).astype(np.float64), S.tpos)


def gpu_fft(dev, Y, So, alpha, **kw):
    g, Z, kl = api.kl_grad_fft(to_dev(Y, dev), sparse_to_dev(So, dev), alpha, want_Z=True, want_kl=True, **kw)
    return g.cpu().numpy().astype(np.float64), Z.item(), kl.item()


# (n, Y std, alpha, p, min_boxes, max_box_width, max_fft)
CASES = [
    (500, 3.0, 12.0, 3, 50, 1.0, 2048),
    (2000, 10.0, 1.0, 2, 20, 0.5, 1024),
    (3001, 20.0, 1.0, 4, 10, 1.0, 2048),
    (4000, 40.0, 1.0, 5, 8, 2.0, 512),      # B capped at max_fft / (2 p) = 51
    (1500, 0.01, 12.0, 3, 50, 1.0, 2048),   # the scale of early iterations: B = min_boxes
    (777, 5.0, 1.0, 3, 1, 0.25, 64),        # the smallest FFT: B = 10, F = 64
]


@pytest.mark.parametrize("case", CASES)
def test_fft_grad_matches_interp_oracle(dev, case):
    n, ystd, alpha, p, mb, mw, mf = case
    say("fft grad vs interp oracle", case)
    _, _, _, S = random_graph_P(n, 30, 10.0, 7)
    So = widen(S)
    Y = synth.random_embedding(n, ystd, 3000 + n)
    g, Z, kl = gpu_fft(dev, Y, So, alpha, n_interp=p, min_boxes=mb, max_box_width=mw, max_fft=mf)
    go, Zo, klo = I.kl_grad(Y, So, alpha, p=p, min_boxes=mb, max_box_width=mw, max_fft=mf)
    e = rel(g, go)
    assert e <= GRAD_RTOL, e
    assert abs(Z - Zo) <= 1e-9 * Zo
    assert abs(kl - klo) <= 1e-5 * max(1.0, abs(klo))


def test_fft_grad_deterministic(dev):
    say("fft grad determinism")
    n = 20_000
    _, _, _, S = random_graph_P(n, 90, 30.0, 2)
    P = sparse_to_dev(widen(S), dev)
    Y = to_dev(synth.random_embedding(n, 15.0, 4100), dev)
    a, Za, _ = api.kl_grad_fft(Y, P, 1.0, want_Z=True)
    b, Zb, _ = api.kl_grad_fft(Y, P, 1.0, want_Z=True)
    assert torch.equal(a, b) and torch.equal(Za, Zb)


def test_fft_grad_same_bits_in_either_row_order(dev):
    """The attraction pass takes the rows in box order unless the KL is asked
    for (then in index order); a row's sum must not depend on which rows
    share its block, so the gradient and Z come out bit for bit the same.
    With k = 90 a block's 16 rows hold about 2,900 entries, so rows straddle
    the 2,048-entry chunks in both orders."""
    say("fft grad: box order vs index order")
    n = 20_000
    _, _, _, S = random_graph_P(n, 90, 30.0, 3)
    P = sparse_to_dev(widen(S), dev)
    Y = to_dev(synth.random_embedding(n, 15.0, 4101), dev)
    a, Za, _ = api.kl_grad_fft(Y, P, 1.0, want_Z=True)
    b, Zb, klb = api.kl_grad_fft(Y, P, 1.0, want_Z=True, want_kl=True)
    assert torch.equal(a, b) and torch.equal(Za, Zb)
    assert torch.isfinite(klb).all()


def test_fft_grad_close_to_exact_c2(dev):
    # the approximation against the exact gradient at 20k points: about 1e-2
    # relative at box side 1 (the method's default), third order below it
    say("fft grad vs exact c2")
    n = 20_000
    _, _, _, S = random_graph_P(n, 90, 30.0, 2)
    P = sparse_to_dev(widen(S), dev)
    for ystd, alpha in ((0.01, 12.0), (20.0, 1.0)):
        Y = to_dev(synth.random_embedding(n, ystd, 4000 + int(ystd)), dev)
        ge, Ze, _, _ = api.kl_grad(Y, P, alpha, want_Z=True)
        ge = ge.cpu().numpy()
        errs = []
        for mw in (1.0, 0.5, 0.25):
            gf, Zf, _ = api.kl_grad_fft(Y, P, alpha, max_box_width=mw, max_fft=4096, want_Z=True)
            errs.append((rel(gf.cpu().numpy(), ge), abs(Zf.item() - Ze.item()) / Ze.item()))
        say("errors vs exact", ystd, errs)
        assert errs[0][0] <= 5e-2 and errs[0][1] <= 2e-3, errs
        assert errs[-1][0] <= 2e-3 and errs[-1][1] <= 1e-4, errs
        if ystd > 1.0:  # (a tiny embedding has B = min_boxes for every width)
            assert errs[-1][0] < errs[0][0] / 8, errs


def test_fft_grad_degenerate(dev):
    say("fft grad degenerate inputs")
    # all points at one position: R = 0, Z = n (n - 1), A = 0
    n = 300
    _, _, _, S = random_graph_P(n, 10, 3.0, 9)
    P = sparse_to_dev(widen(S), dev)
    Y = to_dev(np.full((n, 2), 1.25, np.float32), dev)
    g, Z, kl = api.kl_grad_fft(Y, P, 1.0, want_Z=True, want_kl=True)
    assert torch.isfinite(g).all() and g.abs().max().item() < 1e-6
    assert abs(Z.item() - n * (n - 1)) <= 1e-6 * n * n
    # two points: for P = [[0, 1/2], [1/2, 0]] the attraction and the
    # repulsion cancel up to the interpolation error, so the gradient is a
    # small difference of two terms; compare it on the scale of those terms
    S2 = oracle.CSR(np.array([0, 1, 2]), np.array([1, 0], np.int32), np.array([0.5, 0.5]))
    Y2 = np.array([[0.3, -1.2], [2.0, 0.7]], np.float32)
    g2, Z2, kl2 = api.kl_grad_fft(to_dev(Y2, dev), sparse_to_dev(S2, dev), 1.0, want_Z=True, want_kl=True)
    go, Zo, klo = I.kl_grad(Y2, S2, 1.0)
    scale = 4.0 * np.abs(I.attraction(Y2, S2)).max()
    assert np.abs(g2.cpu().numpy() - go).max() <= 1e-6 * scale
    assert abs(Z2.item() - Zo) <= 1e-9 * Zo


def test_fft_grad_c5_full_size(dev):
    # n = 1,000,000 (the c5 size): the whole repulsion against the oracle of
    # the same scheme, the attraction on a seeded sample of rows against the
    # C oracle's exact sums
    say("fft grad c5")
    n = 1_000_000
    _, _, _, S = random_graph_P(n, 90, 30.0, 5)
    So = widen(S)
    Y = synth.random_embedding(n, 30.0, 2005)
    g, Z, _ = gpu_fft(dev, Y, So, 1.0)
    Ro, Zo = I.repulsion(Y)
    assert abs(Z - Zo) <= 1e-9 * Zo
    rows = np.random.default_rng(5).choice(n, 192, replace=False)
    _, _, Ao = oracle.grad_rows(Y.astype(np.float64), rows, So)
    go = 4.0 * (Ao - Ro[rows] / Zo)
    e = rel(g[rows], go)
    assert e <= GRAD_RTOL, e


def test_fft_grad_clustered_embedding(dev):
    # 95% of 200,000 points in one tight cluster, the rest spread: most
    # points share a few boxes, whose node sums are split into chunks
    say("fft grad clustered")
    n = 200_000
    _, _, _, S = random_graph_P(n, 30, 10.0, 17)
    So = widen(S)
    rng = np.random.default_rng(18)
    Y = np.where(rng.random((n, 1)) < 0.95, rng.normal(0.0, 0.01, (n, 2)), rng.normal(0.0, 20.0, (n, 2)))
    Y = Y.astype(np.float32)
    g, Z, kl = gpu_fft(dev, Y, So, 1.0)
    go, Zo, klo = I.kl_grad(Y, So, 1.0)
    assert rel(g, go) <= GRAD_RTOL, rel(g, go)
    assert abs(Z - Zo) <= 1e-9 * Zo
    g2, Z2, _ = gpu_fft(dev, Y, So, 1.0)
    assert np.array_equal(g, g2) and Z == Z2


# Every transform size (the passes differ by log2 F mod 3 and by the number of
# rows a block takes), each with the grid at its fullest (N = F / 2) and just
# past the size below (N = F / 4 + p).  Z and the repulsion are FP64 sums on
# both sides (1e-9); the gradient carries FP32 attraction terms.
@pytest.mark.parametrize("F", [64, 128, 256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("full", [True, False])
def test_fft_grad_every_transform_size(dev, F, full):
    say("fft grad transform size", F, full)
    n, p = 1201, 2
    _, _, _, S = random_graph_P(n, 10, 3.0, 21)
    So = widen(S)
    Y = synth.random_embedding(n, 4.0, 3100 + F)
    B = F // (2 * p) if full else F // (4 * p) + 1
    kw = dict(min_boxes=B, max_box_width=1e6, max_fft=F)
    g, Z, kl = gpu_fft(dev, Y, So, 1.0, n_interp=p, **kw)
    go, Zo, klo = I.kl_grad(Y, So, 1.0, p=p, **kw)
    assert rel(g, go) <= GRAD_RTOL, rel(g, go)
    assert abs(Z - Zo) <= 1e-9 * Zo
    assert abs(kl - klo) <= 1e-5 * max(1.0, abs(klo))


@pytest.mark.parametrize("p", [2, 3, 4, 5])
def test_fft_grad_box_occupancies(dev, p):
    # boxes holding 1, 15 .. 17 points (the 16 lanes of a box), 63 .. 65 (the
    # points in flight), 255 .. 257 and 511 .. 513 (the chunks of a heavy box)
    say("fft grad box occupancies", p)
    counts = [1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 511, 512, 513, 2049]
    rng = np.random.default_rng(31)
    Y = np.concatenate([[-8.0, 2.0 * (q % 7)] + rng.uniform(0.2, 0.7, (m, 2)) + [2.0 * (q // 7), 0.0]
                        for q, m in enumerate(counts)])
    Y = rng.permutation(np.concatenate([Y, [[-10.0, -10.0], [30.0, 30.0]]])).astype(np.float32)
    _, _, _, S = random_graph_P(Y.shape[0], 10, 3.0, 22)
    So = widen(S)
    kw = dict(min_boxes=40, max_box_width=1.0, max_fft=512)
    g, Z, kl = gpu_fft(dev, Y, So, 1.0, n_interp=p, **kw)
    go, Zo, klo = I.kl_grad(Y, So, 1.0, p=p, **kw)
    assert rel(g, go) <= GRAD_RTOL, rel(g, go)
    assert abs(Z - Zo) <= 1e-9 * Zo


def test_fft_grad_long_rows(dev):
    """The attraction of the box order takes the rows of a block in passes of
    160 entries, and what is longer over the whole block: row lengths around
    the passes' edges and far past them, empty rows and columns outside
    [0, n) (which contribute nothing), in a last block that is not full.  Against the index order, bit for bit,
    and against FP64 sums (an FP32 sum of m terms is within m 2^-24 of the
    terms' absolute sum; the longest row has 7,000)."""
    say("fft grad long rows")
    rng = np.random.default_rng(41)
    n = 8005
    lens = rng.integers(0, 40, n)
    lens[[3, 70, 71, 500, 501, 4000, 4001, 8000, 8004]] = [159, 160, 161, 320, 1023, 1024, 1025, 4097, 7000]
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in lens]).astype(np.int32)
    val = rng.uniform(0.5, 1.5, col.size).astype(np.float32) / np.float32(col.size)
    bad = rng.choice(col.size, 50, replace=False)
    good = np.ones(col.size, bool)
    good[bad] = False
    bcol = col.copy()
    bcol[bad] = rng.choice([-1, n, n + 5, 2**31 - 1], 50)
    P = api.SparseP(to_dev(row_ptr, dev), to_dev(bcol, dev), to_dev(val, dev), None, n)
    Y = synth.random_embedding(n, 8.0, 4200)
    Yd = to_dev(Y, dev)
    a, Za, _ = api.kl_grad_fft(Yd, P, 1.0, want_Z=True)
    b, Zb, _ = api.kl_grad_fft(Yd, P, 1.0, want_Z=True, want_kl=True)
    assert torch.equal(a, b) and torch.equal(Za, Zb)
    Ro, Zo = I.repulsion(Y)
    rows = np.repeat(np.arange(n), lens)[good]
    d = Y[rows].astype(np.float64) - Y[col[good]].astype(np.float64)
    t = (val[good] / (1.0 + (d * d).sum(1)))[:, None] * d
    A, absA = np.zeros((n, 2)), np.zeros((n, 2))
    np.add.at(A, rows, t)
    np.add.at(absA, rows, np.abs(t))
    tol = 4.0 * (lens[:, None] * 2.0**-24 + 1e-6) * absA + 1e-6 * np.abs(4.0 * Ro / Zo) + 1e-12
    err = np.abs(a.cpu().numpy() - 4.0 * (A - Ro / Zo))
    assert (err <= tol).all(), (err / tol).max()


# Rows of a block in passes of 160 entries while half of the rows fill half of
# one, what lies past them flat over the block, 4,096 at a time: all rows at
# the last length without a second pass and the first with one, half of the
# rows long, some, and so many that their ends take several chunks.
@pytest.mark.parametrize("lens", ["240", "241", "half", "some", "many"])
def test_fft_grad_uneven_rows(dev, lens):
    say("fft grad uneven rows", lens)
    rng = np.random.default_rng(43)
    n = 705
    if lens in ("240", "241"):
        m = np.full(n, int(lens))
    else:
        share = {"half": 0.5, "some": 0.05, "many": 0.4}[lens]
        m = np.where(rng.random(n) < share, rng.integers(600, 700, n), rng.integers(0, 40, n))
    row_ptr = np.concatenate([[0], np.cumsum(m)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, q, replace=False)) for q in m]).astype(np.int32)
    val = rng.uniform(0.5, 1.5, col.size).astype(np.float32) / np.float32(col.size)
    P = api.SparseP(to_dev(row_ptr, dev), to_dev(col, dev), to_dev(val, dev), None, n)
    Y = to_dev(synth.random_embedding(n, 8.0, 4300), dev)
    a, Za, _ = api.kl_grad_fft(Y, P, 1.0, want_Z=True)
    b, Zb, _ = api.kl_grad_fft(Y, P, 1.0, want_Z=True, want_kl=True)  # the rows in index order
    assert torch.equal(a, b) and torch.equal(Za, Zb)
