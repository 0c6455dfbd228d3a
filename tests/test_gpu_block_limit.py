"""The largest block the library takes: 2^31 - 1 ratings, all of one cell.  A
position a step past its end no longer fits a signed 32-bit integer, so a loop
that counted in one would wrap and not end.

Every rating is 0 and u.v is exactly 1, so every squared error is exactly 1,
every partial sum an integer below 2^53 and the RMSE exactly 1; a rating left
out or taken twice would change it.

The arrays are untouched zeros, which take next to no host memory until they
are copied; the device holds about 105 GB.  The streamed case is opt-in (set
BGMF_BLOCK_LIMIT=1): 26 GB of pinned host memory and a minute.
"""
import os
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NNZ = 2**31 - 1
T0 = time.time()


def _log(msg):
    print(f"[{time.time() - T0:7.1f} s] {msg}", flush=True)


# U rows in LDS; in global memory; streamed (a ring of two copies of the one
# stratum fits the budget, the one-pass load does not).  k = 16 where one wave
# sums the whole block.
@pytest.mark.parametrize("n,k,budget", [
    pytest.param(40, 64, 0, id="lds"),
    pytest.param(40_000, 16, 0, id="global"),
    pytest.param(40, 16, 40 << 30, id="streamed", marks=pytest.mark.skipif(
        os.environ.get("BGMF_BLOCK_LIMIT") != "1",
        reason="2^31 - 1 streamed ratings: opt in with BGMF_BLOCK_LIMIT=1")),
])
def test_rmse(n, k, budget):
    from paper_2304_13724_amd import bgmf
    rows, cols = np.zeros(NNZ, np.int32), np.zeros(NNZ, np.int32)
    vals = np.zeros(NNZ, np.float32)
    U, V = np.zeros((n, k), np.float32), np.zeros((30, k), np.float32)
    U[:, 0] = V[:, 0] = 1.0
    with bgmf.Model(n, 30, k, 1) as mdl:
        mdl.set_option(bgmf.BGMF_OPT_RATINGS_BUDGET, budget)
        mdl.set_factors(U, V)
        _log("loading")
        mdl.load_coo(rows, cols, vals)
        assert (mdl.get_option(bgmf.BGMF_OPT_STREAM_SLOTS) > 0) == bool(budget)
        _log("loaded")
        r = mdl.rmse()
        _log(f"rmse {r!r} in {mdl.timing()[1]:.0f} ms")
    assert r == 1.0
