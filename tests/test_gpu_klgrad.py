"""GPU parity: tsne_kl_grad (gradient, Z, KL, per-row Z) against the FP64 oracle.

Tolerance: norm-wise relative gradient error 1e-4 (the stated FP32 target),
evaluated at the same float32 Y and P (widened exactly for the oracle).
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import (ROW_RTOL, check_grad_rows, check_step_rows, oracle_problem, random_graph_P, rel, say,
                     sparse_to_dev, to_dev)
from paper_2605_13928_amd import api, synth

pytestmark = pytest.mark.gpu

GRAD_RTOL = 1e-4


def widen(S, v32):
    return oracle.CSR(S.row_ptr, S.col, v32.astype(np.float64), S.tpos)


def compare(dev, S, Y32, alpha, zrow=True):
    v32 = S.val.astype(np.float32)
    So = widen(S, v32)
    P = sparse_to_dev(So, dev)
    g, Z, kl, Zr = api.kl_grad(to_dev(Y32, dev), P, alpha, want_Z=True, want_kl=True, want_Zrow=zrow)
    g = g.cpu().numpy().astype(np.float64)
    go, Zo, klo = oracle.kl_grad(Y32.astype(np.float64), So, alpha)
    e = rel(g, go)
    assert e <= GRAD_RTOL, e
    # and row by row, so that one wrong row cannot hide in the norm
    n = Y32.shape[0]
    check_grad_rows(g, go, Y32.astype(np.float64), np.arange(n), So, alpha, Zo)
    assert abs(Z.item() - Zo) <= 1e-6 * Zo
    assert abs(kl.item() - klo) <= 1e-5 * max(1.0, abs(klo))
    assert np.abs(g.sum(0)).max() <= 1e-5 * np.abs(g).sum()
    if zrow:
        Zro, _, _ = oracle.grad_rows(Y32.astype(np.float64), np.arange(Y32.shape[0]), None)
        np.testing.assert_allclose(Zr.cpu().numpy(), Zro, rtol=1e-6)
    return e


@pytest.mark.parametrize("alpha", [12.0, 1.0])
@pytest.mark.parametrize("ystd", [0.01, 1.0, 30.0])
def test_klgrad_c1(dev, alpha, ystd):
    say("klgrad c1", alpha, ystd)
    X, labels, idx, d2, Pc, S = oracle_problem("c1", 1500, 90, 30.0)
    Y = synth.random_embedding(1500, ystd, 77)
    compare(dev, S, Y, alpha)


# 4161 and 4225 leave 2 and 3 subblocks in the last superblock of 256, so the
# jobs are dealt with the diagonal ones before, resp. after, the jobs against it
@pytest.mark.parametrize("n", [2, 3, 97, 1024, 1025, 4097, 4161, 4225])
def test_klgrad_ragged_sizes(dev, n):
    say("klgrad ragged", n)
    k = min(30, n - 1)
    idx, d2, Pc, S = random_graph_P(n, k, min(10.0, k - 0.5), n)
    Y = synth.random_embedding(n, 5.0, n + 1)
    compare(dev, S, Y, 12.0)


def test_klgrad_two_points_stationary(dev):
    say("klgrad n=2")
    S = oracle.CSR(np.array([0, 1, 2]), np.array([1, 0]), np.array([0.5, 0.5]))
    Y = np.array([[0.3, -1.2], [2.0, 0.7]], np.float32)
    P = sparse_to_dev(S, dev)
    g, Z, kl, _ = api.kl_grad(to_dev(Y, dev), P, 1.0, want_Z=True, want_kl=True)
    assert np.abs(g.cpu().numpy()).max() < 1e-6
    assert abs(kl.item()) < 1e-6


def test_klgrad_c2_full_size(dev):
    # the benchmark's launch configuration: n = 20,000
    say("klgrad c2 full")
    n = 20_000
    idx, d2, Pc, S = random_graph_P(n, 90, 30.0, 2)
    for ystd, alpha in ((0.01, 12.0), (20.0, 1.0)):
        Y = synth.random_embedding(n, ystd, 2000 + int(ystd))
        compare(dev, S, Y, alpha, zrow=False)


# 1,000,000 is the full-scale workload (superblocks of 1024); 49,864 and
# 99,628 (superblocks of 512 and 1024) leave 4 and 5 subblocks in the last
# superblock, which deals the diagonal jobs before the jobs against it.
@pytest.mark.parametrize("n", [49_864, 99_628, 1_000_000])
def test_klgrad_sampled_rows(dev, n):
    # per-row Z_i and gradient rows checked on a seeded sample of rows, plus
    # sum_i Z_i = Z (a property at any size).
    say("klgrad sampled", n)
    idx, d2, Pc, S = random_graph_P(n, 90, 30.0, 5)
    v32 = S.val.astype(np.float32)
    So = widen(S, v32)
    P = sparse_to_dev(So, dev)
    Y = synth.random_embedding(n, 30.0, 2005)
    g, Z, kl, Zr = api.kl_grad(to_dev(Y, dev), P, 1.0, want_Z=True, want_Zrow=True)
    Zr = Zr.cpu().numpy()
    Zg = Z.item()
    assert abs(Zr.sum() - Zg) <= 1e-9 * Zg
    rows = np.random.default_rng(5 + n).choice(n, 192, replace=False)
    Zo, Ro, Ao = oracle.grad_rows(Y.astype(np.float64), rows, So)
    np.testing.assert_allclose(Zr[rows], Zo, rtol=1e-6)
    # g_i = 4 (A_i - R_i / Z) with the oracle's A_i, R_i; Z from the checked row sums
    go = 4.0 * (Ao - Ro / Zg)
    e = rel(g.cpu().numpy()[rows], go)
    assert e <= GRAD_RTOL, e
    check_grad_rows(g.cpu().numpy()[rows], go, Y.astype(np.float64), rows, So, 1.0, Zg)


def test_fused_attraction_full_scale(dev):
    # n = 1,000,000: 977 superblocks, so the bucketing of P's entries by job
    # takes its opposite superblocks in more than one LDS window (the graph
    # is the one of the sampled-rows test above, still cached)
    fused_first_iteration(dev, 1_000_000, 5)


@pytest.mark.parametrize("n", [20_000, 49_864, 50_000, 99_628, 100_003])
def test_fused_attraction_first_iteration(dev, n):
    # tsne_optimize sums the attraction inside the all-pairs kernel (one
    # launch configuration per superblock size: 256, 512 (49,864, 50,000),
    # 1024 (99,628, 100,003) here; the pairs differ in the dealing order).
    fused_first_iteration(dev, n, 7)


def fused_first_iteration(dev, n, seed):
    # At t = 0 the update is -lr * 0.8 * g exactly up to FP32 rounding, so
    # the gradient is recovered from it and checked row by row against the
    # oracle's A_i, R_i (alpha = 12), with Z from tsne_kl_grad at the same Y.
    say("fused attraction", n)
    idx, d2, Pc, S = random_graph_P(n, 90, 30.0, seed)
    So = widen(S, S.val.astype(np.float32))
    P = sparse_to_dev(So, dev)
    Y = synth.random_embedding(n, 5.0, 3000 + n % 97)
    Yd = to_dev(Y, dev)
    _, Z, _, _ = api.kl_grad(Yd, P, 12.0, want_Z=True)
    Yo = Yd.clone()
    U = torch.zeros_like(Yo)
    G = torch.ones_like(Yo)
    api.optimize(Yo, U, G, P, 0, 1, lr=200.0, exaggeration=12.0)
    g = -U.cpu().numpy().astype(np.float64) / (200.0 * 0.8)
    rows = np.random.default_rng(n).choice(n, 256, replace=False)
    Zo, Ro, Ao = oracle.grad_rows(Y.astype(np.float64), rows, So)
    go = 4.0 * (12.0 * Ao - Ro / Z.item())
    e = rel(g[rows], go)
    assert e <= GRAD_RTOL, e
    # g is recovered from the update, which adds one FP32 rounding of lr 0.8 g
    check_grad_rows(g[rows], go, Y.astype(np.float64), rows, So, 12.0, Z.item())
    # and the step itself: Y + update
    np.testing.assert_array_equal(Yo.cpu().numpy(), (Yd + U).cpu().numpy())


def test_fused_loop_bitwise_reproducible_c2(dev):
    # The job-grouped copy of P is filled through LDS atomics, so the order
    # of the entries inside a job's range changes from call to call; the
    # all-pairs kernel sums them in exact 64-bit fixed point, so two runs
    # of the loop from the same state must agree bit for bit.
    say("fused loop determinism c2")
    n = 20_000
    idx, d2, Pc, S = random_graph_P(n, 90, 30.0, 2)
    P = sparse_to_dev(widen(S, S.val.astype(np.float32)), dev)
    Y0 = to_dev(synth.random_embedding(n, 1e-2, 2024), dev)
    runs = []
    for _ in range(2):
        Y = Y0.clone()
        U = torch.zeros_like(Y)
        G = torch.ones_like(Y)
        api.optimize(Y, U, G, P, 0, 30, lr=200.0, exaggeration=12.0)
        runs.append((Y.cpu(), U.cpu(), G.cpu()))
    for a, b in zip(runs[0], runs[1]):
        assert torch.equal(a, b)


def late_state(n, seed):
    """A mid-run optimiser state: embedding at the late scale, a non-zero
    update and gains spread over [0.01, 3] (seeded draws, float32)."""
    rng = np.random.default_rng(seed)
    Y = synth.random_embedding(n, 15.0, seed)
    U = (rng.standard_normal((n, 2)) * 0.3).astype(np.float32)
    G = rng.uniform(0.01, 3.0, (n, 2)).astype(np.float32)
    G[rng.random((n, 2)) < 0.05] = 0.01  # at the floor
    return Y, U, G


@pytest.mark.parametrize("t", [99, 100, 150])
def test_fused_loop_late_schedule_c2(dev, t):
    # One tsne_optimize iteration at t (99: the last exaggerated one; 100:
    # alpha = 1 and momentum 0.8 from here on; 150: mid-run) from a state
    # with a non-zero update and gains != 1, against oracle.kl_grad +
    # oracle.step at the same state, every row and coordinate.
    say("fused loop late schedule", t)
    n = 20_000
    idx, d2, Pc, S = random_graph_P(n, 90, 30.0, 2)
    So = widen(S, S.val.astype(np.float32))
    P = sparse_to_dev(So, dev)
    Y, U, G = late_state(n, 700 + t)
    Yd, Ud, Gd = to_dev(Y, dev), to_dev(U, dev), to_dev(G, dev)
    api.optimize(Yd, Ud, Gd, P, t, t + 1, lr=200.0, exaggeration=12.0, exaggeration_iters=100,
                 momentum_early=0.5, momentum_late=0.8)
    alpha, mom = oracle.tsne_schedule(t)
    Y64 = Y.astype(np.float64)
    go, Zo, _ = oracle.kl_grad(Y64, So, alpha, want_kl=False)
    Ra, Aa = oracle.grad_rows_scale(Y64, np.arange(n), So)
    tol_g = ROW_RTOL * 4.0 * (alpha * Aa + Ra / Zo)
    amb = check_step_rows(Yd.cpu().numpy(), Ud.cpu().numpy(), Gd.cpu().numpy(), Y, U, G, go, tol_g, 200.0, mom)
    assert amb <= 2 * n * 1e-3, amb


# Up to 5,600 points a workgroup takes one pair of 128-point superblocks:
# around the edges of its 64-point subblocks, and around 5,600; above it the
# 256-point superblocks, with 1, 2 and 3 subblocks in the last one (the order
# the jobs are dealt in changes between the latter two).
@pytest.mark.parametrize("n", [5, 63, 64, 65, 127, 128, 129, 191, 193, 257, 5600, 5601, 5633, 5697, 5761])
@pytest.mark.parametrize("zrow", [True, False])
def test_klgrad_small_superblock_edges(dev, n, zrow):
    say("klgrad small superblocks", n, zrow)
    k = min(30, n - 1)
    _, _, _, S = random_graph_P(n, k, min(10.0, k - 0.5), n)
    compare(dev, S, synth.random_embedding(n, 5.0, n + 2), 3.0, zrow)


@pytest.mark.parametrize("n", [5, 64, 129, 1500, 5600, 5601])
def test_fused_attraction_small(dev, n):
    # the fused launches of the same sizes, every row (see fused_first_iteration)
    say("fused attraction small", n)
    k = min(90, n - 1)
    _, _, _, S = random_graph_P(n, k, min(30.0, k - 0.5), 11)
    So = widen(S, S.val.astype(np.float32))
    P = sparse_to_dev(So, dev)
    Y = synth.random_embedding(n, 3.0, 3100 + n)
    runs = []
    for _ in range(2):
        Yo = to_dev(Y, dev)
        U, G = torch.zeros_like(Yo), torch.ones_like(Yo)
        api.optimize(Yo, U, G, P, 0, 1, lr=200.0, exaggeration=12.0)
        runs.append((Yo, U))
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
    go, Zo, _ = oracle.kl_grad(Y.astype(np.float64), So, 12.0)
    g = -runs[0][1].cpu().numpy().astype(np.float64) / (200.0 * 0.8)
    assert rel(g, go) <= GRAD_RTOL
    check_grad_rows(g, go, Y.astype(np.float64), np.arange(n), So, 12.0, Zo)
