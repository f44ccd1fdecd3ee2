"""The work a user has this framework do, as measurable cases.

Every case is one call (or the two calls that belong together) through the
public Python entry points of ``paper_2103_00405_amd.api``:

  simulate     an ensemble of one network, all outputs (``simulate``)
  gradient     an ensemble and the score gradient of a final count
               (``simulate`` + ``score_grad``)
  expectation  the differentiable expectation, forward and backward
               (``expectation`` under torch.autograd)
  batch        many uneven networks in one captured launch (``Batch.run``)

Networks are the catalog's Lotka-Volterra and birth-death models and the
random networks of ``workloads.random_network``; sizes follow the
configurations of ``workloads`` and ``bench.py``, with odd sizes among them.
The network's structure belongs to the case (``net_seed``); initial counts
and the stream's seed come from the inputs' seed.
"""
import math

import numpy as np
import torch

from paper_2103_00405_amd import api
from paper_2103_00405_amd import workloads as W

RANDOM_TIME, DIRECT, LAZY, DIRECT_TREE = 0, 1, 2, 3


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # one small ensemble, as a user explores a model interactively (the
        # catalog's small configuration): a few wavefronts, so the latency of
        # a firing and of the launch decide
        dict(name="lv_small", path="simulate", net="lv", c=1.0, x0=100, t_end=20.0, G=201,
             R=256, method=RANDOM_TIME, breaks=0),
        # the ensemble-throughput configuration (the paper's model)
        dict(name="lv_ensemble", path="simulate", net="lv", c=10.0, x0=1000, t_end=5.0, G=101,
             R=1 << 20, method=RANDOM_TIME, breaks=0),
        # the same model by the comparison method, at the trajectory count of
        # the gradient configuration (fewer trajectories than the device holds)
        dict(name="lv_direct", path="simulate", net="lv", c=10.0, x0=1000, t_end=5.0, G=101,
             R=1 << 18, method=DIRECT, breaks=0),
        # time-dependent rates, a ragged number of trajectories
        dict(name="lv_schedule", path="simulate", net="lv", c=10.0, x0=1000, t_end=2.5, G=33,
             R=100003, method=RANDOM_TIME, breaks=4),
        # sensitivities by automatic differentiation (the gradient
        # configuration): short trajectories, forward and backward
        dict(name="bd_expectation", path="expectation", k1=50.0, k2=1.0, t_end=2.0, R=1 << 18),
        # a small pathway of seven reactions, many trajectories
        dict(name="random_m7", path="simulate", net="random", M=7, N=5, net_seed=35, firings=4000,
             G=51, R=50000, method=RANDOM_TIME, breaks=0),
        # a mid-size network with its score gradient
        dict(name="gradient_m45", path="gradient", M=45, N=11, net_seed=6, firings=2000, G=21,
             R=20000),
        # a network of some hundred reactions
        dict(name="random_m301", path="simulate", net="random", M=301, N=75, net_seed=6,
             firings=20000, G=101, R=4000, method=RANDOM_TIME, breaks=0),
        # the large-network configuration in its three forms
        dict(name="large_eager", path="simulate", net="random", M=4000, N=1000, net_seed=3,
             firings=100000, G=101, R=512, method=RANDOM_TIME, breaks=0),
        dict(name="large_lazy", path="simulate", net="random", M=4000, N=1000, net_seed=3,
             firings=100000, G=101, R=512, method=LAZY, breaks=0),
        dict(name="large_tree", path="simulate", net="random", M=4000, N=1000, net_seed=3,
             firings=100000, G=101, R=512, method=DIRECT_TREE, breaks=0),
        # a screen over many uneven networks (the batched configuration's
        # recipe, fewer of them), replayed from its captured graph
        dict(name="batch_192", path="batch", nets=192, net_seed=4, m_lo=3, m_hi=2048,
             firings=8000, G=101, R=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, no dearer than the dearest listed one."""
    kind = rng.choice(["lv", "lv", "direct", "schedule", "expectation", "thread", "gradient",
                       "mid", "large", "large", "batch"])
    if kind in ("lv", "direct", "schedule"):
        x0 = _log_int(rng, 30, 1000)
        c = x0 / 100.0                      # the fixed point stays at (x0, x0)
        R = _log_int(rng, 64, 1 << 18)
        # 3 c x0 firings per unit of time and trajectory
        t_end = rng.uniform(0.3, 1.0) * min(20.0, 1.5e5 / (3.0 * c * x0))
        return dict(path="simulate", net="lv", c=c, x0=x0, t_end=t_end, G=_log_int(rng, 1, 201),
                    R=R, method=DIRECT if kind == "direct" else RANDOM_TIME,
                    breaks=rng.randint(1, 6) if kind == "schedule" else 0)
    if kind == "expectation":
        return dict(path="expectation", k1=rng.uniform(20.0, 60.0), k2=rng.uniform(0.5, 1.5),
                    t_end=rng.uniform(0.5, 2.0), R=_log_int(rng, 1000, 1 << 18))
    if kind == "gradient":
        M = _log_int(rng, 9, 128)
        return dict(path="gradient", M=M, N=max(2, M // 4), net_seed=rng.randrange(1 << 20),
                    firings=_log_int(rng, 500, 2000), G=_log_int(rng, 1, 51),
                    R=_log_int(rng, 500, 20000))
    if kind == "batch":
        return dict(path="batch", nets=rng.randint(48, 160), net_seed=rng.randrange(1 << 20),
                    m_lo=3, m_hi=_log_int(rng, 600, 2048), firings=_log_int(rng, 2000, 8000),
                    G=_log_int(rng, 11, 101), R=rng.randint(17, 64))
    if kind == "thread":
        M, R, firings = rng.randint(3, 8), _log_int(rng, 256, 50000), _log_int(rng, 500, 4000)
        N = rng.randint(2, 8)
    elif kind == "mid":
        M, R, firings = _log_int(rng, 9, 512), _log_int(rng, 64, 4000), _log_int(rng, 1000, 20000)
        N = max(2, M // 4)
    else:
        M, R, firings = _log_int(rng, 513, 4000), _log_int(rng, 64, 512), _log_int(rng, 5000, 50000)
        N = max(2, M // 4)
    method = RANDOM_TIME
    if kind == "large":
        method = rng.choice([RANDOM_TIME, LAZY, DIRECT_TREE])
    return dict(path="simulate", net="random", M=M, N=N, net_seed=rng.randrange(1 << 20),
                firings=firings, G=_log_int(rng, 1, 201), R=R, method=method, breaks=0)


# ------------------------------------------------------------------ the inputs
def _random_inputs(M, N, net_seed, firings, seed):
    """The recipe of the large and batched configurations: x0 uniform on
    {0..500}, t_end for about `firings` firings at the initial total rate."""
    net = W.random_network(N, M, np.random.default_rng(net_seed))
    x0 = np.random.default_rng(seed).integers(0, 501, size=N).astype(np.int32)
    a0 = W.initial_total_rate(net, x0)
    return net, x0, (float(firings / a0) if a0 > 0 else 1.0)


def _inputs(case, seed):
    """Host inputs: (network spec, x0, t_end, schedule or None, max_firings)."""
    if case["path"] == "expectation":
        rng = np.random.default_rng(seed)
        c = np.array([case["k1"], case["k2"]]) * rng.uniform(0.95, 1.05, size=2)
        return W.birth_death(*c), np.array([0], np.int32), case["t_end"], None, 10_000_000
    if case["path"] == "gradient" or case["net"] == "random":
        net, x0, t_end = _random_inputs(case["M"], case["N"], case["net_seed"], case["firings"],
                                        seed)
        # a network whose rates grow with its state is stopped, as the batched
        # configuration does
        return net, x0, t_end, None, 4 * case["firings"]
    rng = np.random.default_rng(seed)
    net = W.lotka_volterra((case["c"], 0.01, case["c"]))
    lo, hi = int(0.98 * case["x0"]), int(math.ceil(1.02 * case["x0"]))
    x0 = rng.integers(lo, hi + 1, size=2).astype(np.int32)
    sched = None
    if case["breaks"]:
        # every piece scales all rates by one factor around 1
        times = np.linspace(0.0, case["t_end"], case["breaks"] + 2)[1:-1]
        scale = np.array([1.2, 0.8, 1.1, 0.9])[np.arange(case["breaks"]) % 4]
        sched = (times, scale[:, None] * np.asarray(net.c)[None, :])
    return net, x0, case["t_end"], sched, 10_000_000


def _stream_seed(seed):
    return (seed * 2654435761 + 97) & (2 ** 63 - 1)


def prepare(case, seed):
    st = dict(case=case, seed=_stream_seed(seed))
    if case["path"] == "batch":
        rng = np.random.default_rng(case["net_seed"])
        ratio = math.log(case["m_hi"] / case["m_lo"])
        jobs = []
        for i in range(case["nets"]):
            M = int(round(case["m_lo"] * math.exp(rng.uniform(0.0, ratio))))
            spec, x0, t_end = _random_inputs(M, max(2, M // 4), int(rng.integers(1 << 30)),
                                             case["firings"], seed * 4096 + i)
            # (the networks above 256 channels in the lazy form, as the bench)
            jobs.append(dict(net=api.Network(spec), x0=x0, t_end=t_end,
                             sample_t=W.uniform_grid(t_end, case["G"]), R=case["R"],
                             method=LAZY if M > 256 else RANDOM_TIME, net_id=i))
        st["batch"] = api.Batch(jobs, max_firings=5 * case["firings"])
        return st
    spec, x0, t_end, sched, cap = _inputs(case, seed)
    st["net"] = api.Network(spec)
    if sched is not None:
        st["net"].set_schedule(*sched)
    st["x0"] = torch.as_tensor(x0).cuda()
    st["t_end"], st["cap"] = t_end, cap
    if case["path"] == "expectation":
        st["log_c"] = torch.log(torch.as_tensor(np.asarray(spec.c, dtype=np.float64)))
        return st
    st["grid"] = torch.as_tensor(W.uniform_grid(t_end, case["G"])).cuda()
    return st


def _first_count(x_final):
    return x_final[:, 0]


def run(st):
    case = st["case"]
    if case["path"] == "batch":
        # the screen's results gathered into one array per kind, as a program
        # that stores or reduces them does
        st["batch"].run(seed=st["seed"], stats=False)
        outs = st["batch"].outputs
        return {k: torch.cat([o[k].reshape(-1) for o in outs]) for k in sorted(outs[0])}
    if case["path"] == "expectation":
        log_c = st["log_c"].detach().requires_grad_(True)
        value = api.expectation(log_c, st["net"], _first_count, st["x0"], st["t_end"], case["R"],
                                seed=st["seed"])
        value.backward()
        return {"value": value.detach(), "grad": log_c.grad}
    out = api.simulate(st["net"], st["x0"], st["t_end"], st["grid"], case["R"], seed=st["seed"],
                       max_firings=st["cap"], method=case.get("method", RANDOM_TIME), stats=False)
    if case["path"] == "gradient":
        out["grad"], out["se"] = api.score_grad(_first_count(out["x_final"]).to(torch.float64),
                                                out["n"], out["T"])
    return out


# -------------------------------------------------------------- work and truth
def _expected_firings(case):
    """Firings of one trajectory, from the case's own numbers."""
    if case["path"] == "expectation":
        return 2.0 * case["k1"] * case["t_end"]
    if case["path"] in ("gradient", "batch") or case["net"] == "random":
        return float(case["firings"])
    return 3.0 * case["c"] * case["x0"] * case["t_end"]


def _out_bytes(M, N, G, method):
    """Outputs of one trajectory: samples, n, x_final, t_last, status and, for
    the random-time forms, T and tie_step."""
    b = 4 * G * N + 4 * M + 4 * N + 8 + 1
    return b if method in (DIRECT, DIRECT_TREE) else b + 8 * M + 4


def work(case):
    """Arithmetic per firing, the same for every implementation of the method:
    one counter-based random block (60 integer operations), one logarithm to
    binary64 (30), and 5 operations for every channel that has to be looked at
    -- all of them in the eager form, about 20 dependents in the forms that
    follow the dependency graph."""
    if case["path"] == "batch":
        ratio = math.log(case["m_hi"] / case["m_lo"])
        M = (case["m_hi"] - case["m_lo"]) / ratio          # the mean channel count
        R = case["nets"] * case["R"]
        return {"bytes": R * _out_bytes(M, M / 4, case["G"], RANDOM_TIME),
                "flops": R * case["firings"] * (90 + 5 * 20.0)}
    R = case["R"]
    f = _expected_firings(case)
    if case["path"] == "expectation":
        return {"bytes": 8.0 * 5, "flops": R * f * (90 + 5 * 2.0)}
    if case["path"] == "simulate" and case["net"] == "lv":
        M, N = 3, 2
    else:
        M, N = case["M"], case["N"]
    method = case.get("method", RANDOM_TIME)
    touched = min(M, 20) if method in (LAZY, DIRECT_TREE) else M
    b = R * _out_bytes(M, N, case["G"], method) + 8 * case["G"] + 4 * N + 24 * M
    if case["path"] == "gradient":
        b += 16 * M
    return {"bytes": float(b), "flops": R * f * (90 + 5.0 * touched)}


_U32 = 0xFFFFFFFF


def _mulhilo(a, b):
    """High and low 32 bits of a * b for 32-bit values held in int64."""
    lo, hi = a * (b & 0xFFFF), a * (b >> 16)
    top = (hi + (lo >> 16)) >> 16
    return top & _U32, (((hi & 0xFFFF) << 16) + lo) & _U32


def _exponentials(traj, k, block, seed):
    """-ln u of draws 2 block and 2 block + 1 of channel k (Philox4x32-10 at
    counter (block, k, trajectory, 0)), two float64 tensors."""
    x, y, z = torch.broadcast_tensors(block, k, traj)
    w = torch.zeros_like(x)
    k0, k1 = seed & _U32, (seed >> 32) & _U32
    for _ in range(10):
        h0, l0 = _mulhilo(x, 0xD2511F53)
        h1, l1 = _mulhilo(z, 0xCD9E8D57)
        x, y, z, w = h1 ^ y ^ k0, l1, h0 ^ w ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & _U32, (k1 + 0xBB67AE85) & _U32
    even = ((y << 21) | (x >> 11)) + 1
    odd = ((w << 21) | (z >> 11)) + 1
    return -torch.log(even.double() * 2.0 ** -53), -torch.log(odd.double() * 2.0 ** -53)


def _reference(spec, x0, t_end, seed, R, cap):
    """The random-time method (internal clocks, argmin of the gaps) over R
    trajectories side by side, in plain float64 torch operations; returns the
    final counts, n, T and the time of the last firing."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    N, M = spec.N, spec.M
    order = np.zeros((M, 2), np.int64)            # reactant columns; column N holds ones
    order[:] = N
    pair = np.zeros(M, bool)
    nu = np.zeros((M, N), np.int64)
    for k in range(M):
        at = 0
        for e in range(spec.react_ptr[k], spec.react_ptr[k + 1]):
            j, s = int(spec.react_species[e]), int(spec.react_sigma[e])
            order[k, at] = j
            at += 1
            pair[k] |= s == 2
            nu[k, j] -= s
        for e in range(spec.prod_ptr[k], spec.prod_ptr[k + 1]):
            nu[k, int(spec.prod_species[e])] += int(spec.prod_mult[e])
    s0, s1 = (torch.as_tensor(order[:, q], device=dev) for q in (0, 1))
    pair = torch.as_tensor(pair, device=dev)
    nu = torch.as_tensor(nu, device=dev)
    c = torch.as_tensor(np.asarray(spec.c, dtype=np.float64), device=dev)
    X = torch.ones((R, N + 1), dtype=torch.int64, device=dev)
    X[:, :N] = torch.as_tensor(x0, device=dev).long()
    traj = torch.arange(R, device=dev)
    ks = torch.arange(M, device=dev)

    def rates():
        u, v = X[:, s0], X[:, s1]
        h = torch.where(pair, u * (u - 1) // 2, u * v)
        return c * h.double()

    chunk = 32                                    # draws of every channel, made in blocks
    def table(first):
        even, odd = _exponentials(traj[:, None, None], ks[None, :, None],
                                  torch.arange(first // 2, (first + chunk) // 2, device=dev), seed)
        return torch.stack((even, odd), -1).reshape(R, M, chunk)

    draws = table(0)
    P = draws[:, :, 0].clone()
    T = torch.zeros((R, M), dtype=torch.float64, device=dev)
    n = torch.zeros((R, M), dtype=torch.int64, device=dev)
    t = torch.zeros(R, dtype=torch.float64, device=dev)
    alive = torch.ones(R, dtype=torch.bool, device=dev)
    inf = torch.full((), math.inf, dtype=torch.float64, device=dev)
    a, fired, ready = rates(), 0, chunk
    while fired < cap:
        gap = torch.where(a == 0, inf, torch.clamp((P - T) * (1.0 / a), min=0.0))
        d, mu = gap.min(dim=1)
        alive = alive & (t + d <= t_end)
        if fired % 16 == 0 and not bool(alive.any()):
            break
        dz = torch.where(alive, d, 0.0)
        hit = (ks == mu[:, None]) & alive[:, None]
        T = torch.where(hit, P, T + a * dz[:, None])
        n += hit
        if fired % 16 == 0 and int(n.max()) + 18 > ready:
            draws = torch.cat((draws, table(ready)), 2)
            ready += chunk
        E = torch.gather(draws, 2, n[:, :, None])[:, :, 0]
        P = torch.where(hit, P + E, P)
        X[:, :N] += torch.where(alive[:, None], nu[mu], 0)
        t = t + dz
        a = rates()
        fired += 1
    if fired >= cap:
        return None
    T = T + a * (t_end - t)[:, None]
    return X[:, :N], n, T, t


def _score(f, n, T):
    R = f.numel()
    base = (f.sum() - f) / (R - 1)
    y = (f - base)[:, None] * (n.double() - T)
    return y.mean(0), y.std(0) / math.sqrt(R)


def exact(case, seed):
    """Internal times, last event times and score gradients of the shorter
    ensembles; the other outputs are counts."""
    steps = _expected_firings(case)
    if case["path"] == "batch" or case.get("breaks") or case.get("method", 0) != RANDOM_TIME:
        return None
    if steps > 8000 or case["R"] * steps * (case.get("M", 3) + 20) > 4e9:
        return None
    spec, x0, t_end, _, cap = _inputs(case, seed)
    got = _reference(spec, x0, t_end, _stream_seed(seed), case["R"], min(cap, 10000))
    if got is None:                                # a trajectory met the firing cap
        return None
    X, n, T, t_last = got
    f = X[:, 0].double()
    if case["path"] == "expectation":
        return {"value": f.mean(), "grad": _score(f, n, T)[0]}
    out = dict(samples=None, n=None, T=T, x_final=None, t_last=t_last, status=None, tie_step=None)
    if case["path"] == "gradient":
        out["grad"], out["se"] = _score(f, n, T)
    return out
