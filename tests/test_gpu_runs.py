"""Runs in the sweep with V in global memory: 32 or more consecutive ratings
of one row or one column in a block take a step that keeps that row of U or V
in registers.  Its arithmetic is the general step's, so the result is compared
bit for bit with the LDS-staged sweep's general step: run lengths at the edges of the run rule, of its chunks of 16 and of the window
that finds runs, duplicate ratings at every distance inside a run (a row
prefetched 16 ratings ahead would be stale), runs next to each other, to
other ratings and to the block's ends.
"""
import numpy as np
import pytest

from helpers import gpu_run
from workloads.synth import Workload, init_factors

pytestmark = pytest.mark.gpu

LDS, GLOBAL = 1, 2


def _workload(rows, cols, k, p, seed):
    rows, cols = np.asarray(rows, np.int32), np.asarray(cols, np.int32)
    n, m = max(int(rows.max()) + 1, p), max(int(cols.max()) + 1, p)
    vals = np.random.default_rng(seed).integers(1, 6, rows.size).astype(np.float32)
    U0, V0 = init_factors(n, m, k, seed + 1)
    return Workload("runs", n, m, k, p, 0.01, 0.05, 1, rows, cols, vals, U0, V0)


def _same_bits(w, passes=1, **kw):
    a = gpu_run(w, 2, v_staging=LDS, single=0, passes=passes)
    g = gpu_run(w, 2, v_staging=GLOBAL, passes=passes, **kw)
    assert np.array_equal(g[0], a[0]) and np.array_equal(g[1], a[1])


def _block(by_row, length, before, after, dup, at=None):
    """One block: `before` single ratings, a run of `length`, `after` single
    ratings.  `dup`: the run's partner repeats `dup` ratings later, once, in a
    run of a row from rating `at` of the run (a third into it)."""
    rng = np.random.default_rng(1000 * length + dup)
    rows, cols = [], []
    for i in range(before):
        rows.append(i)
        cols.append(int(rng.integers(0, 90)))
    if by_row:
        part = rng.permutation(90)[: min(length, 90)]
        part = np.r_[part, rng.permutation(200)[: length - part.size] + 90]
        if dup and dup < length:
            if at is None:
                at = length // 3 if length // 3 + dup < length else 0
            part[at + dup] = part[at]
        rows += [before] * length
        cols += [int(x) for x in part]
        top = before + 1
    else:
        step = np.ones(length, int)
        if dup:  # in a column run only neighbours can share a row
            step[length // 2] = 0
        rows += [int(x) for x in before + np.cumsum(step)]
        cols += [37] * length
        top = before + length + 1
    for i in range(after):
        rows.append(top + i)
        cols.append(int(rng.integers(0, 90)))
    return rows, cols


@pytest.mark.parametrize("by_row", [True, False], ids=["row", "col"])
@pytest.mark.parametrize("length", [31, 32, 33, 47, 48, 49, 63, 64, 65, 97, 200])
def test_run_lengths(by_row, length):
    for before, after in [(0, 0), (0, 16), (3, 0), (16, 1), (17, 40)]:
        rows, cols = _block(by_row, length, before, after, 0)
        _same_bits(_workload(rows, cols, 64, 1, length + before))


@pytest.mark.parametrize("k", [16, 80, 128, 256])
def test_run_widths(k):
    for by_row in (True, False):
        rows, cols = _block(by_row, 70, 5, 9, 0)
        _same_bits(_workload(rows, cols, k, 1, k))


@pytest.mark.parametrize("dup", [1, 2, 7, 14, 15, 16, 17, 30, 31, 33])
def test_duplicates_in_a_run(dup):
    for k in (32, 128):
        rows, cols = _block(True, 100, 2, 5, dup)
        _same_bits(_workload(rows, cols, k, 1, dup))
    rows, cols = _block(False, 60 + dup, 2, 5, 1)
    _same_bits(_workload(rows, cols, 64, 1, dup))


@pytest.mark.parametrize("at", [0, 1, 14, 15, 16, 17, 30, 31])
def test_duplicates_where_a_run_starts(at):
    """Around the two chunks of 16 in which a duplicate refuses the run."""
    for dup in (1, 8, 15, 16, 17):
        rows, cols = _block(True, 70, 0, 3, dup, at)
        _same_bits(_workload(rows, cols, 64, 1, at + dup))


@pytest.mark.parametrize("passes", [2, 3])
@pytest.mark.parametrize("k", [64, 128])
def test_several_passes(passes, k):
    """A pass starts again from rows the one before stored: after a run that
    ends with the block, before one that starts it, and with a duplicate that
    ends one."""
    for by_row in (True, False):
        for length, before, after, dup in ((64, 0, 0, 0), (64, 5, 0, 0), (70, 0, 9, 0),
                                           (97, 16, 3, 7 if by_row else 1)):
            rows, cols = _block(by_row, length, before, after, dup)
            _same_bits(_workload(rows, cols, k, 1, length + passes), passes=passes)


@pytest.mark.parametrize("schedule", [0, 2])
def test_heavy_users_and_items(schedule):
    """Several blocks, each with a heavy user and a heavy item among other
    ratings: one launch per stratum, which has runs, and the persistent
    schedule, which has none; two passes per block too, and the ratings
    streamed."""
    rng = np.random.default_rng(5)
    n, m, p = 600, 400, 4
    rows = np.r_[np.repeat([10, 310], m), np.tile(np.arange(n), 2), rng.integers(0, n, 1500)]
    cols = np.r_[np.tile(np.arange(m), 2), np.repeat([7, 250], n), rng.integers(0, m, 1500)]
    order = rng.permutation(rows.size)
    w = _workload(rows[order], cols[order], 64, p, 9)
    _same_bits(w, schedule=schedule)
    _same_bits(w, schedule=schedule, passes=2)
    _same_bits(w, schedule=schedule, budget=20_000)


def _epoch_ms(kind, k, schedule=0):
    """Best of eight epochs over 16 x 16 blocks, every fourth column-block
    filled with blocks of 2,000 ratings: of one row and 8 columns, or of runs
    of 8 ratings."""
    from paper_2304_13724_amd import bgmf
    p, width, length = 16, 2048, 2000
    rng = np.random.default_rng(3)
    rows, cols = [], []
    for R in range(p):
        for C in range(0, p, 4):
            dup = kind == "duplicates"
            rows.append((np.zeros(length, int) if dup else np.arange(length) // 8) + R * width)
            cols.append((rng.integers(0, 8, length) if dup else rng.permutation(width)[:length])
                        + C * width)
    last = p * width - 1
    w = _workload(np.r_[np.concatenate(rows), last], np.r_[np.concatenate(cols), last], k, p, 7)
    with bgmf.Model(w.n, w.m, w.k, w.p) as mdl:
        mdl.set_option(bgmf.BGMF_OPT_V_STAGING, GLOBAL)
        mdl.set_option(bgmf.BGMF_OPT_SCHEDULE, schedule)
        mdl.set_factors(w.U0, w.V0)
        mdl.load_coo(w.rows, w.cols, w.vals)
        times = []
        for _ in range(8):
            mdl.epoch(1e-4, 0.05)
            mdl.sync()
            times.append(mdl.timing()[0])
    return min(times)


def test_duplicates_keep_the_general_pace():
    """Blocks full of duplicate ratings have no run to sweep and take as long
    as blocks of the same length without runs: looking for one costs 1%, one
    entered and left again at every chunk cost 40%."""
    duplicates, single = _epoch_ms("duplicates", 64), _epoch_ms("single", 64)
    print(duplicates, single, flush=True)
    assert duplicates <= 1.15 * single


def test_blocks_without_runs_keep_their_pace():
    """Looking for runs costs blocks that have none little: against the
    persistent schedule, whose step is the same without the look, 2% at k =
    128 (a full look at every chunk cost 11%)."""
    looking, plain = _epoch_ms("single", 128), _epoch_ms("single", 128, schedule=2)
    print(looking, plain, flush=True)
    assert looking <= 1.07 * plain
