"""stats.slow_logs: the draws a run's trajectories took whose logarithm needed
the accurate phase, each counted once.

The expected count comes from the run's own firing counts: every draw E(k, n),
n = 0 .. n_k, is made again by the library's Philox and -ln(u) hooks, and those
that took the accurate phase (about one in 2^20) are counted; the thread
mapping also has the next draw of each channel at hand.  The count depends
neither on the launch shape nor on which trajectories share a wavefront."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2103_00405_amd import workloads as W

pytestmark = pytest.mark.gpu

CHUNK = 1 << 24


def _p(t):
    return C.c_void_p(t.data_ptr())


def _slow(ctr, words, seed):
    """Draws (word pairs `words` of the blocks at counters ctr [count, 4]) that
    took the accurate phase."""
    from paper_2103_00405_amd._lib import check, lib
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    n = ctr.shape[0]
    w = torch.empty((n, 4), dtype=torch.int32, device="cuda")
    check(lib().rtssa_debug_philox(_p(ctr), seed & 0xFFFFFFFF, seed >> 32, _p(w), n, stream))
    w = torch.gather(w, 1, torch.stack([words, words + 1], 1)).to(torch.int64) & 0xFFFFFFFF
    m = ((w[:, 1] << 21) | (w[:, 0] >> 11)).contiguous()
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    slow = torch.zeros(n, dtype=torch.uint8, device="cuda")
    check(lib().rtssa_debug_neglog(_p(m), _p(out), _p(slow), n, 0, stream))
    torch.cuda.synchronize()
    return int(slow.sum(dtype=torch.int64))


def _expected(counts, seed, net_id, direct, ahead):
    """counts [R, M]: firings per channel; ahead: draws made past the last one
    taken."""
    total = 0
    counts = counts.to(torch.int64)
    per = (counts.sum(1, keepdim=True) if direct else counts) + 1 + ahead   # draws n = 0 .. count + ahead
    R, M = per.shape
    rows = max(1, int(CHUNK // max(1, int(per.sum(1).max()))))
    for r0 in range(0, R, rows):
        p = per[r0:r0 + rows].reshape(-1)
        at = torch.repeat_interleave(torch.arange(p.numel(), device="cuda"), p)
        n = torch.arange(at.numel(), device="cuda") - (torch.cumsum(p, 0) - p)[at]
        traj, k = r0 + at // M, at % M
        ctr = torch.empty((at.numel(), 4), dtype=torch.int32, device="cuda")
        ctr[:, 0] = (n if direct else n >> 1).to(torch.int32)
        ctr[:, 1] = -1 if direct else k.to(torch.int32)
        ctr[:, 2] = traj.to(torch.int32)
        ctr[:, 3] = net_id
        words = torch.zeros_like(n) if direct else 2 * (n & 1)
        total += _slow(ctr, words, seed)
    return total


def _run(spec, x0, t_end, R, seed, **kw):
    from paper_2103_00405_amd import api
    net = api.Network(spec)
    if "schedule" in kw:
        net.set_schedule(*kw.pop("schedule"))
    g = api.simulate(net, x0, t_end, [t_end], R, seed=seed, net_id=5, want=("n", "status"), **kw)
    torch.cuda.synchronize()
    return g


def _check(spec, x0, t_end, R, seed, least, shapes, **kw):
    for shape in shapes:
        g = _run(spec, x0, t_end, R, seed, **shape, **kw)
        assert int((g["status"] == 2).sum()) == 0
        want = _expected(g["n"], seed, 5, kw.get("method", 0) in (1, 3),
                         1 if g["stats"]["mapping"] == 1 else 0)
        assert want >= least
        assert g["stats"]["slow_logs"] == want, shape


def test_thread_mapping_short_trajectories():
    """Some 150 firings a trajectory: most passes of a wavefront are repeated
    because a trajectory of another lane ends in them."""
    _check(W.birth_death(50.0, 1.0), np.array([20], np.int32), 1.5, 200000, 3, 5,
           [dict(), dict(block=64, grid=300), dict(mapping=2, block=4)])


def test_thread_mapping_schedule_and_firing_cap():
    spec = W.lotka_volterra((1.0, 0.01, 1.0))
    times = np.linspace(0.1, 1.9, 19)
    rates = np.where(np.arange(19) % 2, 1.5, 0.7)[:, None] * np.asarray(spec.c)
    _check(spec, np.array([100, 100], np.int32), 2.0, 30000, 4, 3,
           [dict(), dict(block=128), dict(mapping=2, block=8), dict(mapping=3, block=64)],
           schedule=(times, rates))
    _check(spec, np.array([100, 100], np.int32), 2.0, 60000, 4, 3,
           [dict(max_firings=217), dict(max_firings=217, mapping=2, block=16)])


@pytest.mark.parametrize("method", [1, 3])
def test_direct_methods(method):
    shapes = [dict(), dict(grid=64)]
    _check(W.birth_death(50.0, 1.0), np.array([20], np.int32), 1.5, 100000, 7, 3, shapes,
           method=method)
    spec = W.lotka_volterra((1.0, 0.01, 1.0))
    _check(spec, np.array([100, 100], np.int32), 2.0, 60000, 8, 3,
           [dict(max_firings=f) for f in (191,)], method=method)


@pytest.mark.parametrize("M", [7, 45, 200])
def test_random_networks_every_mapping(M):
    rng = np.random.default_rng(50 + M)
    spec = W.random_network(max(2, M // 4), M, rng, logc=(-1.0, 1.0), bimol_scale=0.02)
    x0 = rng.integers(5, 40, size=spec.N).astype(np.int32)
    t_end = 300 / W.initial_total_rate(spec, x0)
    shapes = [dict(), dict(mapping=2, block=32), dict(mapping=3, block=64), dict(method=2)]
    _check(spec, x0, t_end, 60000, 9, 5, shapes, max_firings=2000)
