"""GPU parity: tsne_pca (randomized truncated SVD on the FP32 matrix cores)
against the FP64 oracle of the same method (oracle/pca.py) on the same X and
the same test matrix Omega: singular values, the mean, the leading
components and scores; orthonormal components and scores = Xc V^T at any
size; bitwise reproducible."""
import numpy as np
import pytest
import torch

from helpers import say, to_dev
from oracle import pca as opca
from paper_2605_13928_amd import api, synth

pytestmark = pytest.mark.gpu


def run(dev, X, k, Om, q):
    sc, comp, sv, mu = api.pca(to_dev(X, dev), k, to_dev(Om, dev), q)
    return sc.cpu().numpy().astype(np.float64), comp.cpu().numpy().astype(np.float64), sv.cpu().numpy(), \
        mu.cpu().numpy().astype(np.float64)


# (n, g, k, q, latent scale range); ragged n and g against the 128-row and
# 32 / 64-column tiles
CASES = [
    (5000, 300, 50, 2, (100.0, 1.0)),
    (4099, 129, 10, 0, (50.0, 5.0)),
    (1000, 64, 64, 1, (20.0, 2.0)),
    (20011, 517, 32, 2, (100.0, 0.5)),
]


@pytest.mark.parametrize("case", CASES)
def test_pca_matches_oracle(dev, case):
    n, g, k, q, (top, bottom) = case
    say("pca vs oracle", case)
    X = synth.make_expression(n, g, 7 + n, latent=min(64, g), top=top, bottom=bottom)
    Om = synth.make_omega(g, 11 + g)
    sc, comp, sv, mu = run(dev, X, k, Om, q)
    osc, ocomp, osv, omu = opca.randomized_pca(X.astype(np.float64), k, Om.astype(np.float64), q)
    np.testing.assert_allclose(mu, omu, rtol=1e-5, atol=1e-5)
    # singular values: well conditioned, to FP32 accuracy relative to the largest
    assert np.abs(sv - osv).max() <= 2e-5 * osv[0], (sv[:4], osv[:4])
    # components and scores: FP32 rounding in the products is ~3e-6 s_1, so a
    # component's angle error is ~3e-6 s_1 / (gap s_c); checked where the
    # relative gap to both neighbours is >= 2 % and s_c >= 0.05 s_1
    gap = np.minimum(np.abs(np.diff(np.r_[np.inf, osv])), np.abs(np.diff(np.r_[osv, 0.0]))) / osv
    good = np.where((gap[:k] > 0.02) & (osv[:k] >= 0.05 * osv[0]))[0]
    assert good.size >= min(k, 4)
    dots = np.sum(comp[good] * ocomp[good], axis=1)
    assert np.all(dots > 1 - 1e-4), dots.min()
    col_err = np.linalg.norm(sc[:, good] - osc[:, good], axis=0) / np.linalg.norm(osc[:, good], axis=0)
    assert col_err.max() <= 1e-2 and col_err[0] <= 1e-4, col_err
    # properties at any size
    np.testing.assert_allclose(comp @ comp.T, np.eye(k), atol=2e-5)
    # scores = Xc V^T holds as far as Q spans the range of Xc: the GPU's
    # deviation from it matches the oracle's
    Xd = X.astype(np.float64)
    proj = (Xd - mu) @ comp.T
    oproj = (Xd - omu) @ ocomp.T
    dg = np.linalg.norm(sc - proj) / np.linalg.norm(proj)
    do = np.linalg.norm(osc - oproj) / np.linalg.norm(oproj)
    assert dg <= do + 1e-4, (dg, do)
    for c in range(k):
        assert comp[c, np.argmax(np.abs(comp[c]))] > 0


def test_pca_deterministic(dev):
    say("pca determinism")
    X = to_dev(synth.make_expression(30000, 700, 3), dev)
    Om = to_dev(synth.make_omega(700, 4), dev)
    a = api.pca(X, 50, Om, 2)
    b = api.pca(X, 50, Om, 2)
    assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_pca_cells_full_size(dev):
    # 200,000 cells x 2,000 genes (the c3 cell count): full parity with the
    # oracle on the singular values and leading components
    say("pca 200k x 2000")
    n, g, k = 200_000, 2000, 50
    X = synth.make_expression(n, g, 2024)
    Om = synth.make_omega(g, 2025)
    sc, comp, sv, mu = run(dev, X, k, Om, 2)
    osc, ocomp, osv, omu = opca.randomized_pca(X.astype(np.float64), k, Om.astype(np.float64), 2)
    assert np.abs(sv - osv).max() <= 2e-5 * osv[0]
    dots = np.sum(comp[:20] * ocomp[:20], axis=1)
    assert np.all(dots > 1 - 1e-6), dots.min()
    rows = np.random.default_rng(1).choice(n, 2000, replace=False)
    e = np.linalg.norm(sc[rows, :20] - osc[rows, :20]) / np.linalg.norm(osc[rows, :20])
    assert e <= 1e-4, e


def test_pca_rank_deficient(dev):
    # X of rank 5 (plus the offset): the 64-column subspace is rank 5, its
    # Gram matrix singular -- the shifted first CholeskyQR pass must carry
    # it; the 5 nonzero singular values and their components match the
    # oracle, the rest are ~0, and everything stays finite and orthonormal
    say("pca rank 5")
    n, g, k = 3000, 200, 10
    X = synth.make_expression(n, g, 41, latent=5, top=50.0, bottom=5.0, noise=0.0)
    Om = synth.make_omega(g, 42)
    sc, comp, sv, mu = run(dev, X, k, Om, 2)
    osc, ocomp, osv, omu = opca.randomized_pca(X.astype(np.float64), k, Om.astype(np.float64), 2)
    assert np.isfinite(sc).all() and np.isfinite(comp).all() and np.isfinite(sv).all()
    np.testing.assert_allclose(sv[:5], osv[:5], rtol=1e-4)
    assert np.all(sv[5:] <= 1e-3 * sv[0]), sv
    dots = np.abs(np.sum(comp[:5] * ocomp[:5], axis=1))
    assert np.all(dots > 1 - 1e-4), dots
    np.testing.assert_allclose(comp @ comp.T, np.eye(k), atol=1e-3)


# The splits: fewer tiles of 128 rows than fill the chip (their columns are
# split, down to the smallest n and g), one tile past a whole round of 512
# (split) and a round and a half (not split), row chunks of 64 rows and more.
# Tolerances as in test_pca_matches_oracle; the spectrum falls by 1.13 per
# component, so every gap is at least 8 %.
@pytest.mark.parametrize("n,g,k", [(64, 64, 5), (129, 65, 8), (300, 1000, 20), (2700, 1838, 20), (65_537, 70, 12),
                                   (98_400, 68, 12)])
def test_pca_split_sizes(dev, n, g, k):
    say("pca split sizes", n, g, k)
    X = synth.make_expression(n, g, 70 + n, latent=min(64, g), top=100.0, bottom=0.05)
    Om = synth.make_omega(g, 71 + g)
    sc, comp, sv, mu = run(dev, X, k, Om, 2)
    osc, ocomp, osv, omu = opca.randomized_pca(X.astype(np.float64), k, Om.astype(np.float64), 2)
    np.testing.assert_allclose(mu, omu, rtol=1e-5, atol=1e-5)
    assert np.abs(sv - osv).max() <= 2e-5 * osv[0]
    gap = np.minimum(np.abs(np.diff(np.r_[np.inf, osv])), np.abs(np.diff(np.r_[osv, 0.0]))) / osv
    good = np.where((gap[:k] > 0.02) & (osv[:k] >= 0.05 * osv[0]))[0]
    assert good.size >= 4
    assert np.all(np.sum(comp[good] * ocomp[good], axis=1) > 1 - 1e-4)
    np.testing.assert_allclose(comp @ comp.T, np.eye(k), atol=2e-5)
    sc2, comp2, _, _ = run(dev, X, k, Om, 2)
    assert np.array_equal(sc, sc2) and np.array_equal(comp, comp2)


@pytest.mark.parametrize("bottom", [1.0, 1e-2, 1e-4])
def test_pca_steep_spectra(dev, bottom):
    # 64 factors falling over up to six decades below the largest: the single
    # CholeskyQR passes between the products and the one-sided Jacobi method
    # meet condition numbers up to what FP32 data can hold
    say("pca steep spectrum", bottom)
    n, g, k = 3000, 400, 20
    X = synth.make_expression(n, g, 81, top=100.0, bottom=bottom, noise=0.0, offset=0.5)
    Om = synth.make_omega(g, 82)
    sc, comp, sv, mu = run(dev, X, k, Om, 2)
    osc, ocomp, osv, omu = opca.randomized_pca(X.astype(np.float64), k, Om.astype(np.float64), 2)
    assert np.abs(sv - osv).max() <= 2e-5 * osv[0]
    good = np.where(osv[:k] >= 0.05 * osv[0])[0]
    assert np.all(np.sum(comp[good] * ocomp[good], axis=1) > 1 - 1e-4)
    np.testing.assert_allclose(comp @ comp.T, np.eye(k), atol=2e-5)


def test_pca_low_rank(dev):
    # rank 20: the directions past it are not defined, the 20 leading ones are
    say("pca low rank")
    rng = np.random.default_rng(83)
    n, g, r = 2000, 300, 20
    X = (rng.standard_normal((n, r)) * np.geomspace(10.0, 2.0, r)) @ np.linalg.qr(rng.standard_normal((g, r)))[0].T
    X = np.ascontiguousarray(X, dtype=np.float32)
    sc, comp, sv, mu = run(dev, X, r, synth.make_omega(g, 84), 2)
    U, s, Vt = np.linalg.svd(X.astype(np.float64) - X.astype(np.float64).mean(0), full_matrices=False)
    assert np.abs(sv - s[:r]).max() <= 2e-5 * s[0]
    assert np.all(np.abs(np.sum(comp * Vt[:r], axis=1)) > 1 - 1e-4)
    np.testing.assert_allclose(comp @ comp.T, np.eye(r), atol=2e-5)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_pca_non_finite_input(dev, bad):
    # one such entry makes its column's mean, and with it every product with
    # X, NaN: the call returns NaN and no comparison that is false for NaN
    # leaves an index at a value outside the matrices
    say("pca non-finite", bad)
    n, g, k = 1000, 300, 20
    X = synth.make_expression(n, g, 91)
    X[123, 45] = bad
    sc, comp, sv, mu = run(dev, X, k, synth.make_omega(g, 92), 2)
    assert np.isnan(sc).all() and np.isnan(comp).all()
    assert not np.isfinite(mu[45]) and np.isfinite(np.delete(mu, 45)).all()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_pca_non_finite_input_uses_nothing_stale(dev, bad):
    # the eigenvalues' places are a permutation for NaN too: every singular
    # value is written, and no output depends on what the workspace held
    say("pca non-finite, workspace", bad)
    n, g, k = 500, 128, 64
    X = synth.make_expression(n, g, 93)
    X[7, 3] = bad
    Xd, Om = to_dev(X, dev), to_dev(synth.make_omega(g, 94), dev)
    ws = api.Workspace()
    api.pca(to_dev(synth.make_expression(n, g, 95), dev), k, Om, 2, ws=ws)  # sizes it, leaves finite numbers in it
    for fill in (None, 0, 0x3F):
        if fill is not None:
            ws.buf.fill_(fill)
        sc, comp, sv, _ = api.pca(Xd, k, Om, 2, ws=ws)
        assert torch.isnan(sv).all() and torch.isnan(comp).all() and torch.isnan(sc).all()


@pytest.mark.parametrize("rows", [1, 2, 5, 20, 63])
def test_pca_few_distinct_rows(dev, rows):
    # `rows` distinct cells, repeated (1: a constant X): equal rows stay equal
    # bit for bit in every product, so the 64 columns of the subspace are
    # exactly dependent and the Gram matrices' last pivots are zero or
    # rounding errors of either sign.  Rank rows - 1 after centring: those
    # components and values as of the dense SVD, the rest zero or rounding
    # (the mean's, 6e-8 of the entries, over sqrt(n)).
    say("pca few distinct rows", rows)
    rng = np.random.default_rng(96 + rows)
    n, g = 700, 96
    r = rows - 1
    k = max(r, 1)
    X = (3.0 * rng.standard_normal((rows, g)) + 1.0)[np.arange(n) % rows].astype(np.float32)
    sc, comp, sv, mu = run(dev, X, k, synth.make_omega(g, 97), 2)
    assert np.isfinite(sc).all() and np.isfinite(comp).all() and np.isfinite(sv).all()
    if r == 0:
        assert np.all(sv <= 1e-4) and np.all(np.abs(sc) <= 1e-4)
        return
    U, s, Vt = np.linalg.svd(X.astype(np.float64) - X.astype(np.float64).mean(0), full_matrices=False)
    assert np.abs(sv - s[:r]).max() <= 2e-5 * s[0], (sv, s[:r])
    # spans instead of vectors: neighbouring values may be close
    np.testing.assert_allclose(comp.T @ (comp @ Vt[:r].T), Vt[:r].T, atol=1e-3)
    np.testing.assert_allclose(comp @ comp.T, np.eye(r), atol=1e-3)
    np.testing.assert_allclose(sc @ comp, (U[:, :r] * s[:r]) @ Vt[:r], atol=1e-3 * s[0] / np.sqrt(n))
