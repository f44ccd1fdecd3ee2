"""Selection in binary32 keys against the oracle over the rates' whole range.

The thread, sub-wave and workgroup kernels order the gaps (P - T) / a in binary32 and fall
back to the exact selection where that order cannot decide.  Scaling every rate
by f and the times by 1 / f moves gaps and propensities through binary32's
normal range, past it and into its subnormals; every output stays bit-exact.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_00405_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = (("samples", None), ("n", np.uint32), ("T", np.uint64), ("x_final", None),
        ("t_last", np.uint64), ("status", None), ("seq_hash", np.uint64), ("tie_step", np.uint32))


def _compare(spec, x0, t_end, grid, R, seed, **kw):
    from paper_2103_00405_amd import api
    g = api.simulate(api.Network(spec), x0, t_end, grid, R, seed=seed, with_hash=True, **kw)
    torch.cuda.synchronize()
    ref = oracle.simulate(spec, x0, t_end, grid, seed, R)
    for key, view in KEYS:
        got, want = g[key].cpu().numpy(), ref[key]
        if view is not None:
            got, want = got.view(view), want.view(view)
        assert np.array_equal(got, want), key
    for key in ("firings", "near_ties", "clamps", "status_count"):
        assert g["stats"][key] == ref["stats"][key], key
    return ref


def _net(M, seed):
    rng = np.random.default_rng(seed)
    N = max(2, M // 4)
    spec = W.random_network(N, M, rng, logc=(-1.0, 1.0), bimol_scale=0.02)
    x0 = rng.integers(5, 40, size=N).astype(np.int32)
    a0 = W.initial_total_rate(spec, x0)
    return spec, x0, 150.0 / a0


def _mapping(lanes):
    """block and mapping of a lane count: 0 automatic, <= 64 sub-wave, else workgroup."""
    return dict(block=lanes, **({"mapping": 2 if lanes <= 64 else 3} if lanes else {}))


@pytest.mark.parametrize("M,lanes", [(5, 0), (40, 8), (100, 16), (300, 64), (700, 128),
                                     (1100, 256)])
@pytest.mark.parametrize("f", [1e-200, 1e-45, 1e-33, 1e-20, 1e17, 1e40, 1e200])
def test_scaled_rates_bit_exact(M, lanes, f):
    spec, x0, t_end = _net(M, 100 + M)
    spec = W.with_rates(spec, np.asarray(spec.c) * f)
    t_end = t_end / f
    ref = _compare(spec, x0, t_end, np.linspace(0.0, t_end, 9), 70, 3, **_mapping(lanes))
    assert ref["stats"]["firings"] > 70 * 30


@pytest.mark.parametrize("M,lanes", [(6, 0), (48, 8), (200, 32), (600, 128)])
def test_channels_far_apart_bit_exact(M, lanes):
    """A third of the channels at 1e-60 and 1e-45 of the others' rates: they hold
    the binary32 form at +inf without being frozen."""
    spec, x0, t_end = _net(M, 200 + M)
    c = np.asarray(spec.c).copy()
    c[::3] *= 1e-60
    c[1::6] *= 1e-45
    _compare(W.with_rates(spec, c), x0, t_end, np.linspace(0.0, t_end, 5), 64, 4,
             **_mapping(lanes))


@pytest.mark.parametrize("lanes", [4, 8, 64])
@pytest.mark.parametrize("slots", [1, 2, 3, 4, 5, 6, 7, 8])
def test_every_slot_count_bit_exact(lanes, slots):
    """Channel counts at both ends of each slot count of the sub-wave mapping."""
    for M in {(slots - 1) * lanes + 1, slots * lanes}:
        spec, x0, t_end = _net(M, 300 + M)
        _compare(spec, x0, t_end, np.linspace(0.0, t_end, 5), 40, 5, mapping=2, block=lanes)
