"""The library's host code without a GPU: which calls it takes, what it
allocates and how it shapes a launch.

Each test runs in a child process in which ``fake_hip.c`` stands for the HIP
runtime (host memory; launches are recorded, no kernel runs), so the entry
points of the built library run as they are."""
import ctypes as C
import json
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

THREAD, WAVE, WORKGROUP = 1, 2, 3
LAZY = 2


# ---- in the child
class Host:
    def __init__(self):
        from paper_2103_00405_amd import _lib
        self.lib, self.types = _lib.lib(), _lib
        self.fake = C.CDLL(os.environ["LD_PRELOAD"])
        self.keep = []

    def counter(self, name, ctype=C.c_int64):
        return ctype.in_dll(self.fake, "fake_" + name)

    def network(self, M, N):
        """k reads species k mod N and turns it into the next one."""
        sp = np.arange(M, dtype=np.int32) % N
        ptr = np.arange(M + 1, dtype=np.int32)
        one = np.ones(max(M, 1), np.int32)
        c = np.ones(max(M, 1))
        arrs = [ptr, sp, one, ptr, ((sp + 1) % N).astype(np.int32), one]
        h = C.c_void_p()
        rc = self.lib.rtssa_network_create(N, M, *[a.ctypes.data for a in arrs], c.ctypes.data,
                                           C.byref(h))
        assert rc == 0, self.error()
        return h

    def error(self):
        return self.lib.rtssa_last_error().decode()

    def simulate(self, net, N, R, entry="rtssa_simulate", **options):
        x0 = np.zeros(N, np.int32)
        opt = self.types.Options(**options)
        return getattr(self.lib, entry)(net, x0.ctypes.data, 0, 1.0, None, 0, 1, 0, 0, R, None,
                                        0, 0, 0, *[None] * 7, C.byref(opt), None, None)

    def batch(self, nets, R):
        """(create's, run's) codes of one batch of (network, species) pairs."""
        items = (self.types.BatchItem * len(nets))()
        for it, (net, N) in zip(items, nets):
            x0 = np.zeros(N, np.int32)
            self.keep.append(x0)
            it.net, it.x0, it.t_end, it.R = net, x0.ctypes.data, 1.0, R
        b = C.c_void_p()
        rc = self.lib.rtssa_batch_create(items, len(nets), None, None, C.byref(b))
        if rc:
            return rc, None
        rc = self.lib.rtssa_batch_run(b, 1, 0, None, None)
        self.lib.rtssa_batch_destroy(b)
        return 0, rc


# ---- in the test process
@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake_hip") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", "-I/opt/rocm/include", "-o", so,
                    os.path.join(HERE, "fake_hip.c")], check=True)
    return so


def _child(fake, body):
    """``body`` (Python statements with the Host as h, leaving `result`) in a
    child process on the fake runtime."""
    code = ("import sys, json\nsys.path[:0] = [%r, %r]\n"
            "from test_host_calls import *\nh = Host()\n%s\n"
            "print('RESULT ' + json.dumps(result), flush=True)\n" % (ROOT, HERE, body))
    p = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, LD_PRELOAD=fake),
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    return json.loads([x for x in p.stdout.splitlines() if x.startswith("RESULT ")][-1][7:])


SUBWAVE_SIZES = [(9, 8), (20, 900), (64, 512), (64, 1900), (64, 3000), (100, 1000), (250, 2000),
                 (300, 700), (512, 2048), (512, 6000)]


@pytest.mark.parametrize("M,N", SUBWAVE_SIZES)
def test_subwave_acceptance_does_not_depend_on_the_trajectories(fake_hip, M, N):
    """The sub-wave mapping's automatic lanes follow the number of trajectories;
    a network that runs with few of them runs with many, alone and in a batch,
    and a workgroup asks for no more LDS than a CU has."""
    got = _child(fake_hip, """
net = h.network(%d, %d)
result = []
for R in (1, 300, 3000, 30000, 300000):
    rc = h.simulate(net, %d, R, mapping=WAVE)
    result.append((rc, h.counter('last_lds').value, h.batch([(net, %d)], R)))
""" % (M, N, N, N))
    for rc, lds, batch in got:
        assert rc == 0 and batch == [0, 0], got
        assert 0 < lds < 160 * 1024 - 6 * 1024


def test_subwave_batch_of_unlike_networks_fits(fake_hip):
    """A class takes its slots from one network and its species from another."""
    got = _child(fake_hip, """
sizes = [(M, N) for M in (17, 30, 33, 40, 41, 48, 49, 64, 65, 100, 128, 200, 256, 300, 384, 400, 512)
         for N in (9, 500, 1500, 2000, 2050, 2100)]
nets = [(h.network(M, N), N) for M, N in sizes]
result = [h.batch(nets, R) for R in (1, 10, 100, 1000, 10000)]
""")
    assert got == [[0, 0]] * 5


def test_subwave_refuses_species_past_the_lds(fake_hip):
    assert _child(fake_hip, """
net = h.network(64, 45000)
result = [(h.simulate(net, 45000, R, mapping=WAVE), h.error()) for R in (1, 30000)]
""") == [[-2, "sub-wave LDS too large"]] * 2


@pytest.mark.parametrize("mapping,method", [(THREAD, 0), (0, 1), (WAVE, 0), (WORKGROUP, 0)])
def test_a_block_below_one_is_the_mapping_s_own(fake_hip, mapping, method):
    got = _child(fake_hip, """
net = h.network(3, 2)
result = [(h.simulate(net, 2, 5000, mapping=%d, method=%d, block=b), h.counter('last_block').value)
          for b in (0, -1, -64, -2147483648)]
""" % (mapping, method))
    assert got == [got[0]] * 4 and got[0][0] == 0


def test_tree_methods_run_without_memory_for_the_records(fake_hip):
    """The tree methods need their rows (about 256 bytes a channel) but not the
    eager mappings' records (2 KiB a channel) built beside them: with memory
    for the rows alone they run, and a call that must not allocate does not try."""
    got = _child(fake_hip, """
net = h.network(400, 100)
limit, mallocs = h.counter('malloc_limit', C.c_size_t), h.counter('mallocs')
limit.value = 400 * 64 * 16
need = C.c_size_t()
opt = h.types.Options(method=LAZY)
result = [h.lib.rtssa_workspace_size(net, 10, C.byref(opt), C.byref(need))]
before = mallocs.value
result.append(h.simulate(net, 100, 1, entry='rtssa_simulate_noalloc', method=LAZY))
ws = np.zeros(need.value + 512, np.uint8)
at = (ws.ctypes.data + 255) // 256 * 256
result.append(h.simulate(net, 100, 10, method=LAZY, workspace=at, workspace_bytes=need.value))
result.append(mallocs.value - before)
result.append(h.simulate(net, 100, 10, mapping=WAVE))      # needs the records
limit.value = 1 << 60
result.append(h.simulate(net, 100, 10, mapping=WAVE))
result.append(h.lib.rtssa_network_destroy(net))
""")
    assert got == [0, 0, 0, 0, -4, 0, 0]


@pytest.mark.parametrize("M", [9, 200, 512])
def test_subwave_rows_are_one_allocation_and_one_copy(fake_hip, M):
    assert _child(fake_hip, """
net = h.network(%d, 40)
mallocs, copies = h.counter('mallocs').value, h.counter('copies').value
opt, need = h.types.Options(mapping=WAVE), C.c_size_t()
result = [h.lib.rtssa_workspace_size(net, 10, C.byref(opt), C.byref(need)),
          h.counter('mallocs').value - mallocs, h.counter('copies').value - copies]
""" % M) == [0, 1, 1]


@pytest.mark.parametrize("M,N,lanes,block", [
    (64, 16, 8, 128), (60, 15, 8, 128), (48, 12, 8, 256), (40, 10, 8, 256), (301, 75, 64, 256),
    (64, 400, 8, 192), (250, 1500, 32, 192), (400, 3000, 64, 192), (64, 1900, 8, 128)])
def test_subwave_workgroups_fill_the_lds(fake_hip, M, N, lanes, block):
    """Wavefronts per workgroup: the number that leaves a CU the most of them."""
    assert _child(fake_hip, """
net = h.network(%d, %d)
result = [h.simulate(net, %d, 5000, mapping=WAVE, block=%d), h.counter('last_block').value]
""" % (M, N, N, lanes)) == [0, block]
