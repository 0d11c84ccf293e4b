"""The channel stage's lane merge (grids off the bucket merge: sparse streams
whose time cells widen, and more than 16 die queues per channel) against the
reference model, bit for bit.  The shapes sit where it can go wrong: every
number of lanes per die run (1, 3, 8, 16, 17, 33 and 64 die queues), channel
counts that leave units partly filled or group several windows, loads from
idle to a crowded device, runs longer than a lane group (cells taken in
several steps), ties across dies, cells wider than 2^32 ns, and two calls on
carried clocks."""
import numpy as np
import pytest

from paper_2609_09800_amd import workloads as wl
from test_gpu_parity import run_both, torch  # noqa: F401

pytestmark = pytest.mark.gpu

# (channels, dies, planes, tR, flags): plane-parallel counts dies * planes queues per channel
GEOMS = [(3, 1, 1, 3000, 0), (5, 3, 1, 700, 0), (32, 8, 2, 3000, 0), (40, 16, 1, 3000, 0), (2, 17, 1, 900, 0),
         (7, 11, 3, 3000, 1), (32, 16, 4, 3000, 1), (1, 32, 2, 50, 1)]
# mean gap over the time one page takes of all channels
LOADS = [0.4, 1.1, 6.0, 400.0]


@pytest.mark.parametrize("geo", GEOMS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("load", LOADS)
def test_lane_merge_loads(torch, geo, load):  # noqa: F811
    C, D, P, tR, flags = geo
    params = wl.geometry(C, D, P, t_read_ns=tR, flags=flags)
    w = wl.random_stream(C * 100 + D, 40_001, params, 1 << 16, 2048 / C * load, out_frac=0.05, run_frac=0.4)
    run_both(torch, params, w.ranges, [(w.addr[:30_000], w.issue[:30_000]), (w.addr[30_000:], w.issue[30_000:])],
             f"lane merge {geo} load {load}")


@pytest.mark.parametrize("geo", [(4, 4, 1, 3000, 0), (16, 16, 1, 3000, 0), (4, 16, 4, 1000, 1), (2, 13, 1, 2000, 0)],
                         ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("quiet", [10**6, 10**9, 10**14])
def test_lane_merge_crowded_cells(torch, geo, quiet):  # noqa: F811
    """Bursts of thousands of simultaneous requests (equal die-done times on
    every die) between quiet stretches that widen the cells: up to past 2^32
    ns, where die-order entries are no longer packed, and past 2^30 ns, where
    one step cannot span a cell."""
    C, D, P, tR, flags = geo
    params = wl.geometry(C, D, P, t_read_ns=tR, flags=flags)
    rng = np.random.default_rng(quiet % 97 + C)
    issue = np.concatenate([np.sort(rng.integers(0, 50, 6000)) + k * quiet for k in range(5)]).astype(np.int64)
    addr = np.uint64(1 << 40) + rng.integers(0, 1 << 14, issue.size).astype(np.uint64) * np.uint64(16384)
    run_both(torch, params, [(1 << 40, 16384 << 14)], [(addr, issue), (addr[:7000], issue[:7000] + 5 * quiet)],
             f"crowded {geo} quiet {quiet}")


@pytest.mark.parametrize("geo", [(8, 64, 1, 3000, 0), (4, 16, 1, 3000, 0), (2, 3, 1, 3000, 0)],
                         ids=lambda g: "x".join(map(str, g)))
def test_lane_merge_hot_queues_in_a_sparse_stream(torch, geo):  # noqa: F811
    """Wide cells that a few crowded die queues make too big for one step:
    steps end at the queues' lanes, at the cell's end, and with ties across
    dies at the step's end."""
    C, D, P, tR, flags = geo
    params = wl.geometry(C, D, P, t_read_ns=tR, flags=flags)
    rng = np.random.default_rng(C)
    n = 30_000
    issue = np.sort(rng.integers(0, n * 40_000 // C, n))
    issue[10_000:14_000] = issue[10_000]          # simultaneous: ties on every die
    page = rng.integers(0, 1 << 14, n)
    hot = rng.random(n) < 0.3
    page[hot] = page[hot] // (C * D) * (C * D) + C * rng.integers(0, 2, int(hot.sum()))
    addr = np.uint64(1 << 40) + page.astype(np.uint64) * np.uint64(16384)
    run_both(torch, params, [(1 << 40, 16384 << 15)], [(addr, issue), (addr[:9_000], issue[:9_000] + issue[-1])],
             f"hot queues {geo}")


def test_lane_merge_long_reads(torch):  # noqa: F811
    """tR near its limit: a cell's minimum width exceeds 2^30 ns."""
    params = wl.geometry(2, 3, 1, t_read_ns=(1 << 29) - 7)
    w = wl.random_stream(4, 9_000, params, 4096, 1e9)
    run_both(torch, params, w.ranges, [(w.addr, w.issue)], "long reads")
