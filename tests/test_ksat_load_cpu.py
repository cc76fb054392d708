"""Loading k-SAT instances on the host: layouts, threads, limits."""
import subprocess
import sys
import time

import numpy as np
import pytest

from paper_2111_13628_amd import instances, nmc

ROOT = __file__.rsplit("/", 2)[0]

FEW_THREADS = """
import ctypes, resource, sys
sys.path.insert(0, {root!r})
from paper_2111_13628_amd import instances, nmc
nmc.lib()
cp, lits = instances.gen_ksat({n}, "9.8", 4, 7)
# stacks of 1 GiB: the address space left has room for {room} of them
libc = ctypes.CDLL(None)
attr = ctypes.create_string_buffer(64)
assert libc.pthread_attr_init(attr) == 0
assert libc.pthread_attr_setstacksize(attr, ctypes.c_size_t(1 << 30)) == 0
assert libc.pthread_setattr_default_np(attr) == 0
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + ({room} << 30) + (900 << 20), -1))
print("loaded", nmc.Instance.ksat({n}, cp, lits).info.n_items)
"""


@pytest.mark.parametrize("n,room", [(300, 0), (5000, 0), (5000, 2), (30000, 0), (30000, 3)])
def test_load_with_few_threads(n, room):
    """Records are placed by several threads from some size on; with room for
    none or only a few of them, the threads there are do all of the work."""
    r = subprocess.run([sys.executable, "-c", FEW_THREADS.format(root=ROOT, n=n, room=room)], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0 and f"loaded {n}" in r.stdout, (r.returncode, r.stderr[-500:])


@pytest.mark.parametrize("n", [1, 3])
def test_reads_ahead_stay_inside(n):
    """The sweeps read a whole block of 8 slots (256 + 4 x 1024 bytes), the split
    sweeps six rows of 1024 bytes, from the last chunk's first one on, however
    few slots the chunk has: both record arrays hold that."""
    cp = np.arange(n + 1, dtype=np.int32)
    inst = nmc.Instance.ksat(n, cp, np.arange(1, n + 1, dtype=np.int32))
    per_class = 256 + 1024 + 1024  # the shortest chunk in either layout
    assert inst.footprint(1)[0] >= 256 + 4 * 1024 + 6 * 1024 + per_class


def test_split_layout_only_where_it_fits():
    """Classes of 150 variables: up to 9,500 variables the split layout is a
    second set of records beside the sweep layout's; at 10,000 no split sweep
    fits in LDS, so there is none, as at 13,000."""

    def per_variable(n):
        cp, lits = instances.gen_ksat(n, "9.8", 4, n)
        return nmc.Instance.ksat(n, cp, lits, 150).footprint(1)[0] / n

    large = per_variable(13000)
    assert per_variable(9500) > 1.2 * large
    assert per_variable(10000) < 1.05 * large


def test_load_cost(monkeypatch):
    """What placing the records by LDS bank adds to a load, in CPU time of all
    threads: four times a load without placement is the limit (measured: 2.2
    times; placing one address order at a time 6.2 times for two layouts, 4.5
    times for one)."""
    cp, lits = instances.gen_ksat(20000, "9.8", 4, 5)

    def cpu_s():
        best = np.inf
        for _ in range(4):
            t = time.process_time()
            nmc.Instance.ksat(20000, cp, lits)
            best = min(best, time.process_time() - t)
        return best

    placed = cpu_s()
    monkeypatch.setenv("NMC_KSAT_BANK_SCHEDULE", "0")
    unplaced = cpu_s()
    assert placed < 4 * unplaced, (placed, unplaced)
