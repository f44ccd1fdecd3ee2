"""The sub-wave mapping's automatic lane counts against the CPU oracle.

The lanes of a trajectory follow from the network and the number of
trajectories; every choice gives the same bits, and a network with many
species runs at any number of trajectories."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_00405_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = (("samples", None), ("n", np.uint32), ("T", np.uint64), ("x_final", None),
        ("t_last", np.uint64), ("status", None), ("seq_hash", np.uint64), ("tie_step", np.uint32))


def _net(M, N, seed, firings):
    rng = np.random.default_rng(seed)
    spec = W.random_network(N, M, rng, logc=(-1.0, 1.0), bimol_scale=0.02)
    x0 = rng.integers(5, 40, size=N).astype(np.int32)
    return spec, x0, firings / W.initial_total_rate(spec, x0)


def _equal(g, ref, rows, keys=KEYS):
    for key, view in keys:
        got, want = g[key][rows].cpu().numpy(), ref[key]
        if view is not None:
            got, want = got.view(view), want.view(view)
        assert np.array_equal(got, want), key


@pytest.mark.parametrize("M,N,R,lanes", [
    (45, 11, 300, 64), (45, 11, 2000, 32), (45, 11, 3000, 16), (45, 11, 9001, 8),
    (20, 5, 30000, 8), (100, 25, 3000, 16), (200, 50, 2000, 32), (301, 75, 2000, 64),
    # species that need more lanes than the channels, or most of a CU's LDS
    (64, 512, 300, 64), (64, 512, 30000, 8), (100, 1000, 3000, 16), (64, 3000, 9000, 32)])
def test_automatic_lanes_bit_exact(M, N, R, lanes):
    from paper_2103_00405_amd import api
    spec, x0, t_end = _net(M, N, 400 + M, 60)
    grid = np.array([0.4, 1.0]) * t_end
    g = api.simulate(api.Network(spec), x0, t_end, grid, R, seed=8, mapping=2, with_hash=True)
    torch.cuda.synchronize()
    assert g["stats"]["block"] == lanes
    for r0, n in ((0, 100), (R // 2, 100), (R - 100, 100)):
        ref = oracle.simulate(spec, x0, t_end, grid, 8, n, traj_offset=r0)
        _equal(g, ref, slice(r0, r0 + n))
    assert sum(g["stats"]["status_count"]) == R
