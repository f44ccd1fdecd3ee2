"""GPU score-function gradient: the backward kernel against the plain numpy
reference, the analytic birth-death derivative, coupled finite differences,
and the autograd wrapper.

Pass bands: each test compares a family of m estimates; every comparison
uses z = Phi^-1(1 - alpha / (2 m)) standard errors with the family-wise
level alpha = 0.01 (Bonferroni), so a correct estimator fails a test with
probability at most 1 %.  The runs are seeded, so a pass is reproducible.
"""
import math

import numpy as np
import pytest
import torch
from scipy import stats

from oracle.score import score_grad as score_ref
from paper_2103_00405_amd import workloads as W

pytestmark = pytest.mark.gpu


def _api():
    from paper_2103_00405_amd import api
    return api


ALPHA = 0.01


def _z(m):
    """Two-sided Bonferroni band for a family of m comparisons at level ALPHA."""
    return float(stats.norm.isf(ALPHA / (2 * m)))


def _analytic_bd(k1, k2, T):
    m = k1 / k2 * (1 - math.exp(-k2 * T))
    dm = np.array([m, -m + k1 * T * math.exp(-k2 * T)])
    return m, dm, (1 + 2 * m) * dm


@pytest.mark.parametrize("baseline", [True, False])
def test_backward_kernel_matches_reference(baseline):
    api = _api()
    rng = np.random.default_rng(1)
    for R, M in ((1, 3), (7, 2), (1000, 5), (70_000, 3), (5000, 300)):
        f = rng.normal(size=R) * 3 + 1
        n = rng.integers(0, 50, size=(R, M)).astype(np.int32)
        T = rng.uniform(0, 50, size=(R, M))
        g, se = api.score_grad(torch.tensor(f, device="cuda"), torch.tensor(n, device="cuda"),
                               torch.tensor(T, device="cuda"), baseline=baseline)
        gr, ser = score_ref(f, n, T, baseline=baseline)
        assert np.allclose(g.cpu().numpy(), gr, rtol=1e-10, atol=1e-12), (R, M)
        if R > 1:
            assert np.allclose(se.cpu().numpy(), ser, rtol=1e-8, atol=1e-12), (R, M)


def test_birth_death_analytic_gradient():
    api = _api()
    w = W.bd_gradient()
    net = api.Network(w.net)
    o = api.simulate(net, w.x0, w.t_end, w.sample_t, w.R, seed=3, want=("x_final", "n", "T"))
    X = o["x_final"][:, 0].to(torch.float64)
    m, dm, dm2 = _analytic_bd(50.0, 1.0, 2.0)
    z = _z(4)                                       # 2 functions x 2 channels
    for f, ref in ((X, dm), (X * X, dm2)):
        g, se = api.score_grad(f, o["n"], o["T"])
        g, se = g.cpu().numpy(), se.cpu().numpy()
        assert np.all(np.abs(g - ref) < z * se), (g, ref, se)
        # the check has power: a zero or sign-flipped gradient would fail it
        assert np.all(np.abs(ref) > 2 * z * se)


def _coupled_fd(api, net, w, c0, k, h, seed, species=0):
    """X_T(species) at c_k e^{+h} and c_k e^{-h} with the same seed and
    trajectory ids (common per-channel streams); species=None: every one."""
    vals = []
    for s in (+1, -1):
        c = c0.copy()
        c[k] *= math.exp(s * h)
        net.set_rates(c)
        o = api.simulate(net, w.x0, w.t_end, w.sample_t, w.R, seed=seed, want=("x_final",))
        x = o["x_final"].to(torch.float64)
        vals.append(x if species is None else x[:, species])
    net.set_rates(c0)
    return vals


def test_coupled_finite_differences_birth_death():
    """Central differences in log c_k with common random streams (same seed and
    trajectory ids) agree with the score estimate and the analytic value, for
    E[X_T] and E[X_T^2]."""
    api = _api()
    w = W.bd_gradient()
    net = api.Network(w.net)
    h = 1e-3
    c0 = np.array(w.net.c)
    base = api.simulate(net, w.x0, w.t_end, w.sample_t, w.R, seed=9, want=("x_final", "n", "T"))
    X = base["x_final"][:, 0].to(torch.float64)
    _, dm, dm2 = _analytic_bd(50.0, 1.0, 2.0)
    z = _z(8)                               # 2 functions x 2 channels x 2 comparisons
    for power, ref in ((1, dm), (2, dm2)):
        g, se = api.score_grad(X ** power, base["n"], base["T"])
        for k in range(2):
            up, down = _coupled_fd(api, net, w, c0, k, h, 9)
            d = (up ** power - down ** power) / (2 * h)
            fd, fd_se = float(d.mean()), float(d.std() / math.sqrt(w.R))
            # central differences carry an O(h^2) bias: 1e-3 relative bounds it here
            assert abs(fd - ref[k]) < z * fd_se + 1e-3 * abs(ref[k]), (power, k, fd, ref[k])
            band = z * math.sqrt(fd_se**2 + float(se[k])**2)
            assert abs(fd - float(g[k])) < band, (power, k)
            assert abs(fd) > 2 * band              # power against a zero estimate


def test_coupled_finite_differences_lotka_volterra():
    """The ensemble model at T = 5: the score estimates of dE[X_j]/dlog c_k and
    dE[X_j^2]/dlog c_k for both species agree with coupled central
    differences within their standard errors (no closed form here).  The
    score's per-path terms (n_k - T_k, T_k ~ 5e4 here) are noisy, so the
    comparison runs 2^21 trajectories: then a zero estimate fails every
    comparison whose finite difference is well away from zero (checked)."""
    api = _api()
    w = W.lv_gradient(R=1 << 21)
    net = api.Network(w.net)
    h = 1e-3
    c0 = np.array(w.net.c)
    base = api.simulate(net, w.x0, w.t_end, w.sample_t, w.R, seed=11, want=("x_final", "n", "T"))
    X = base["x_final"].to(torch.float64)
    fds = [_coupled_fd(api, net, w, c0, k, h, 11, species=None) for k in range(3)]
    z = _z(12)                              # 2 species x 2 functions x 3 channels
    powered = 0
    for j in range(2):
        for power in (1, 2):
            g, se = api.score_grad(X[:, j] ** power, base["n"], base["T"])
            for k in range(3):
                up, down = fds[k]
                d = (up[:, j] ** power - down[:, j] ** power) / (2 * h)
                fd, fd_se = float(d.mean()), float(d.std() / math.sqrt(w.R))
                band = z * math.sqrt(fd_se**2 + float(se[k])**2)
                print("species %d power %d channel %d: fd %.4g +- %.3g, score %.4g +- %.3g, "
                      "band %.3g" % (j, power, k, fd, fd_se, float(g[k]), float(se[k]), band))
                assert abs(fd - float(g[k])) < band, (j, power, k, fd, fd_se, float(g[k]))
                powered += abs(fd) > band
    # a zero gradient would fail most comparisons (those with |fd| beyond the band)
    assert powered >= 10, powered


def test_autograd_expectation():
    """The autograd wrapper returns exactly the backward kernel's estimate on
    the same paths, and that estimate matches the analytic derivative."""
    api = _api()
    w = W.bd_gradient(R=1 << 18)
    net = api.Network(w.net)
    log_c = torch.tensor(np.log(w.net.c), dtype=torch.float64, requires_grad=True)
    f = lambda x: x[:, 0].to(torch.float64)
    loss = api.expectation(log_c, net, f, w.x0, w.t_end, w.R, seed=4)
    loss.backward()
    # the same paths directly
    o = api.simulate(net, w.x0, w.t_end, [w.t_end], w.R, seed=4, want=("x_final", "n", "T"))
    fx = f(o["x_final"])
    assert float(loss.detach()) == float(fx.mean())
    g, se = api.score_grad(fx, o["n"], o["T"])
    assert torch.equal(log_c.grad, g.cpu())
    m, dm, _ = _analytic_bd(50.0, 1.0, 2.0)
    z = _z(3)                                   # the mean and two channels
    assert abs(float(loss.detach()) - m) < z * math.sqrt(m / w.R)
    assert np.all(np.abs(log_c.grad.numpy() - dm) < z * se.cpu().numpy())


@pytest.mark.parametrize("R,M", [(1, 1), (1, 300), (2, 5), (255, 7), (256, 256), (257, 257),
                                 (300, 1000), (5000, 64), (70001, 3), (600000, 2), (9000, 1100)])
def test_score_grad_partitions(R, M):
    """Sizes around the edges of the reduction's partitions: one row, more
    channels than a block's threads, one and many blocks.  Every term is within
    a few ulps and at most about 40 are added in one chain, so 1e-12 of the sum of
    magnitudes bounds the difference to a float64 sum in any order."""
    from paper_2103_00405_amd import api
    gen = torch.Generator().manual_seed(R * 7 + M)
    f = torch.rand(R, dtype=torch.float64, generator=gen) * 10
    n = torch.randint(0, 50, (R, M), dtype=torch.int32, generator=gen)
    T = torch.rand((R, M), dtype=torch.float64, generator=gen) * 50
    g, se = (v.cpu() for v in api.score_grad(f.cuda(), n.cuda(), T.cuda()))
    base = (f.sum() - f) / (R - 1) if R > 1 else torch.zeros_like(f) + f.sum() - f
    y = (f - base)[:, None] * (n.double() - T)
    assert bool(((g - y.mean(0)).abs() <= 1e-12 * y.abs().mean(0) + 1e-300).all())
    if R > 1:
        want = y.std(0) / R ** 0.5
        assert bool(((se - want).abs() <= 1e-9 * want).all())
    else:
        assert not bool(se.any())
