"""Rate schedules where the kernels' forms change, against the CPU oracle: every
slot count of the sub-wave kernel, automatic lane counts, and pieces whose rates
leave the range in which gaps are ordered in binary32 and come back (each kernel
chooses the order anew at a breakpoint)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_00405_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = (("samples", None), ("n", np.uint32), ("T", np.uint64), ("x_final", None),
        ("t_last", np.uint64), ("status", None), ("seq_hash", np.uint64), ("tie_step", np.uint32))


def _net(M, seed, firings):
    rng = np.random.default_rng(seed)
    spec = W.random_network(max(2, M // 4), M, rng, logc=(-1.0, 1.0), bimol_scale=0.02)
    x0 = rng.integers(5, 40, size=spec.N).astype(np.int32)
    return spec, x0, firings / W.initial_total_rate(spec, x0)


def _schedule(spec, t_end, seed):
    rng = np.random.default_rng(seed)
    times = np.array([0.15, 0.4, 0.65, 1.5]) * t_end
    rates = np.asarray(spec.c) * rng.uniform(0.3, 2.0, size=(4, spec.M))
    rates[1, rng.random(spec.M) < 0.3] = 0.0
    return times, rates


def _range_schedule(spec, t_end):
    """Pieces: a third of the rates times 1e-60; the network's own; some of the
    degradations times 1e30; the own; another third times 1e-45; the own."""
    c = np.asarray(spec.c)
    rates = np.repeat(c[None], 6, axis=0)
    rates[0, ::3] *= 1e-60
    first_order = np.array([spec.react_sigma[a:b].sum() == 1 for a, b in
                            zip(spec.react_ptr[:-1], spec.react_ptr[1:])])
    no_product = np.diff(spec.prod_ptr) == 0
    rates[2, np.flatnonzero(first_order & no_product)[:2]] *= 1e30
    rates[4, 1::3] *= 1e-45
    return np.array([0.1, 0.25, 0.4, 0.55, 0.7, 0.85]) * t_end, rates


def _compare(spec, x0, t_end, sched, R, seed, lanes=None, rows=None, **kw):
    from paper_2103_00405_amd import api
    grid = np.linspace(0.0, t_end, 7)
    net = api.Network(spec)
    net.set_schedule(*sched)
    g = api.simulate(net, x0, t_end, grid, R, seed=seed, with_hash=True, **kw)
    torch.cuda.synchronize()
    if lanes is not None:
        assert g["stats"]["block"] == lanes
    n = rows or R
    ref = oracle.simulate(spec, x0, t_end, grid, seed, n, schedule=sched)
    for key, view in KEYS:
        got, want = g[key][:n].cpu().numpy(), ref[key]
        if view is not None:
            got, want = got.view(view), want.view(view)
        assert np.array_equal(got, want), key
    if n == R:
        for key in ("firings", "near_ties", "clamps", "status_count"):
            assert g["stats"][key] == ref["stats"][key], key
    return ref


@pytest.mark.parametrize("lanes", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("slots", [2, 4, 5, 6, 8])
def test_every_slot_count_with_schedule(lanes, slots):
    spec, x0, t_end = _net(slots * lanes, 500 + slots, 400)
    _compare(spec, x0, t_end, _schedule(spec, t_end, 1), 24, 6, mapping=2, block=lanes)


@pytest.mark.parametrize("M,R,lanes", [(45, 300, 64), (45, 2000, 32), (45, 3000, 16),
                                       (45, 9001, 8), (100, 9000, 16)])
def test_automatic_lanes_with_schedule(M, R, lanes):
    spec, x0, t_end = _net(M, 600 + M, 80)
    _compare(spec, x0, t_end, _schedule(spec, t_end, 2), R, 7, lanes=lanes, rows=150, mapping=2)


@pytest.mark.parametrize("M,mapping,block", [
    (5, 1, 0), (8, 1, 64), (20, 2, 4), (40, 2, 8), (100, 2, 16), (300, 2, 64),
    (50, 3, 64), (700, 3, 128), (1100, 3, 256), (5000, 3, 1024)])
def test_rates_leave_the_binary32_range_and_return(M, mapping, block):
    spec, x0, t_end = _net(M, 700 + M, 900)
    ref = _compare(spec, x0, t_end, _range_schedule(spec, t_end), 24, 9, mapping=mapping,
                   block=block)
    assert ref["stats"]["firings"] > 24 * 100


@pytest.mark.parametrize("f", [1e-40, 1e-150, 1e40])
def test_rates_set_later_are_ordered_by_their_own_scale(f):
    """set_rates moves a workgroup-mapping network out of the binary32 range and
    back, alone and under a batch that was made before."""
    from paper_2103_00405_amd import api
    spec, x0, t_end = _net(700, 901, 300)
    c = np.asarray(spec.c)
    net = api.Network(spec)
    job = dict(net=net, x0=x0, t_end=t_end / f, sample_t=[t_end / f], R=8, net_id=0)
    batch = api.Batch([job], max_firings=2000, with_hash=True)
    for scale in (f, 1.0, f):
        net.set_rates(c * scale)
        batch.run(seed=5)
        g = api.simulate(net, x0, t_end / f, [t_end / f], 8, seed=5, with_hash=True,
                         max_firings=2000)
        torch.cuda.synchronize()
        if scale != f:
            continue
        ref = oracle.simulate(W.with_rates(spec, c * scale), x0, t_end / f, [t_end / f], 5, 8,
                              max_firings=2000)
        for key, view in KEYS:
            for out in (g, batch.outputs[0]):
                got, want = out[key].cpu().numpy(), ref[key]
                if view is not None:
                    got, want = got.view(view), want.view(view)
                assert np.array_equal(got, want), key
    batch.close()
