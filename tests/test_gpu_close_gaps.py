"""Two smallest gaps planted close together, against the CPU oracle.

The eager kernels order gaps in binary32 and decide in binary64 where the second
smallest lies within a margin of the smallest (2^-18 in the thread mapping, 2^-12
in the sub-wave mapping, 2^-8 to 2^-15 in the workgroup mapping, by its threads
and slots).  The rates of a network of births put the first gaps of two channels
at g and g (1 + delta), for delta from 0 to 2^-6 of either sign, inside, at and
outside every margin; the pair shares a lane, a wavefront or neither."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_00405_amd import workloads as W

pytestmark = pytest.mark.gpu

DELTAS = [0.0, 2.0**-52, 2.0**-50, 0.9e-12, 1.1e-12, 2.0**-36, 2.0**-30, 2.0**-26]
DELTAS += [2.0**-e * s for e in range(24, 5, -1) for s in (1 - 2.0**-5, 1 + 2.0**-5)]


def _network(M, seed, i, j, delta):
    """Births with first gaps 1 (channel i), 1 + delta (channel j), >= 1.5."""
    rng = np.random.default_rng(seed)
    gap = rng.uniform(1.5, 40.0, size=M)
    gap[i], gap[j] = 1.0, 1.0 + delta
    P = np.array([oracle.exp1(seed, 0, 2, k, 0) for k in range(M)])
    return W.from_reactions(2, [({}, {k % 2: 1}, P[k] / gap[k]) for k in range(M)])


def _pairs(M, lanes):
    """(lower, higher): one lane's slots, neighbouring lanes, far apart."""
    out = [(0, 1), (M // 3, M - 1)]
    if 0 < lanes < M:
        out.append((1, 1 + lanes))
    return out


@pytest.mark.parametrize("M,mapping,lanes", [
    (2, 1, 0), (3, 1, 0), (4, 1, 0), (8, 1, 0), (7, 2, 4), (30, 2, 4), (45, 2, 16), (120, 2, 32),
    (500, 2, 64), (60, 3, 64), (700, 3, 128), (1000, 3, 64), (4000, 3, 256), (3000, 3, 1024)])
def test_close_first_gaps_bit_exact(M, mapping, lanes):
    from paper_2103_00405_amd import api
    x0 = np.zeros(2, np.int32)
    fired = []
    for n, delta in enumerate(DELTAS):
        for i, j in _pairs(M, lanes):
            for a, b in ((i, j), (j, i)):
                spec = _network(M, 40 + n, a, b, delta)
                g = api.simulate(api.Network(spec), x0, 50.0, [1.0, 50.0], 1, seed=40 + n, net_id=2,
                                 mapping=mapping, block=lanes, max_firings=3, with_hash=True)
                torch.cuda.synchronize()
                ref = oracle.simulate(spec, x0, 50.0, [1.0, 50.0], 40 + n, 1, net_id=2,
                                      max_firings=3)
                for key in ("n", "T", "t_last", "seq_hash", "tie_step", "samples"):
                    got = g[key].cpu().numpy()
                    assert np.array_equal(got.view(np.uint8), ref[key].view(np.uint8)), (key, delta, a, b)
                for key in ("near_ties", "clamps", "firings"):
                    assert g["stats"][key] == ref["stats"][key], (key, delta, a, b)
                fired.append(int(ref["stats"]["near_ties"]))
    assert max(fired) >= 1 and min(fired) == 0
