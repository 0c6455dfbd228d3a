"""RMSE kernels at the edges of their wave steps: rating counts around one and
several steps of every width (4 to 64 ratings per step, up to eight steps in
flight), widths that fill their lanes and widths that do not, U rows in LDS
and in global memory, streamed, and over caller-given ratings in host and
device memory.  Reference: dots and squares in binary64; each dot in binary32
is off by at most k roundings of its terms' sizes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ref(rows, cols, vals, U, V):
    d = vals - (U[rows].astype(np.float64) * V[cols]).sum(1)
    return float(np.sqrt((d * d).mean()))


@pytest.mark.parametrize("k", [16, 32, 48, 64, 80, 128, 144, 256])
@pytest.mark.parametrize("n", [40, 40_000])  # 20 rows in LDS; 20,000 do not fit
def test_counts_and_widths(k, n):
    from paper_2304_13724_amd import bgmf  # before torch: one HIP runtime
    import torch
    rng = np.random.default_rng(k + n)
    m, p = 30, 2
    U = rng.standard_normal((n, k)).astype(np.float32)
    V = rng.standard_normal((m, k)).astype(np.float32)
    for nnz in (1, 3, 16, 17, 47, 64, 65, 191, 193, 1_537, 9_001):
        rows = rng.integers(0, n, nnz).astype(np.int32)
        cols = rng.integers(0, m, nnz).astype(np.int32)
        vals = rng.integers(1, 6, nnz).astype(np.float32)
        ref = _ref(rows, cols, vals, U, V)
        # a dot of k terms of size about 1: at most k roundings of sqrt(k),
        # which a wide dot and its error here exceed only in its last bits
        tol = k * 2.0 ** -24 * np.sqrt(k) / max(ref, 1.0) + 1e-7
        with bgmf.Model(n, m, k, p) as mdl:
            mdl.set_factors(U, V)
            mdl.load_coo(rows, cols, vals)
            assert abs(mdl.rmse() - ref) <= tol * ref
            host = mdl.rmse_coo(rows, cols, vals)
            assert abs(host - ref) <= tol * ref
            dev = [torch.from_numpy(a).cuda() for a in (rows, cols, vals)]
            torch.cuda.synchronize()
            assert bgmf.bgmf_rmse_coo_dev(mdl.h, *[t.data_ptr() for t in dev], nnz) == host
        with bgmf.Model(n, m, k, p) as mdl:  # streamed: room for both strata, not for the load
            mdl.set_option(bgmf.BGMF_OPT_RATINGS_BUDGET, 2 * 8 * (nnz + 256) + 64)
            mdl.set_factors(U, V)
            mdl.load_coo(rows, cols, vals)
            assert mdl.get_option(bgmf.BGMF_OPT_STREAM_SLOTS) > 0
            assert abs(mdl.rmse() - ref) <= tol * ref


@pytest.mark.parametrize("k", [16, 32, 48, 64, 128, 256])
def test_many_blocks(k):
    """A grid whose launches take one wave step at a time from k = 48 up
    (p = 1056: 71,808 waves in-core, 16,896 streamed) with U rows too many
    for LDS; the grids above take two."""
    from paper_2304_13724_amd import bgmf
    rng = np.random.default_rng(k)
    p, nnz = 1056, 60_000
    n, m = p * (41_000 // k + 1), p + 7
    U = rng.random((n, k), dtype=np.float32)
    V = rng.random((m, k), dtype=np.float32)
    # half of the ratings in a few blocks, so that some are longer than a step
    rows = np.r_[rng.integers(0, n, nnz // 2), rng.integers(0, 3 * n // p, nnz // 2)].astype(np.int32)
    cols = np.r_[rng.integers(0, m, nnz // 2), rng.integers(0, 6, nnz // 2)].astype(np.int32)
    vals = rng.integers(1, 6, nnz).astype(np.float32)
    ref = _ref(rows, cols, vals, U, V)
    # a dot is about k / 4 with at most k roundings of its size
    tol = k * 2.0 ** -24 * (k / 4) / ref
    got = []
    for budget in (0, 2 << 20):
        with bgmf.Model(n, m, k, p) as mdl:
            mdl.set_option(bgmf.BGMF_OPT_RATINGS_BUDGET, budget)
            mdl.set_factors(U, V)
            mdl.load_coo(rows, cols, vals)
            assert (mdl.get_option(bgmf.BGMF_OPT_STREAM_SLOTS) > 0) == bool(budget)
            got.append(mdl.rmse())
            assert abs(got[-1] - ref) <= tol * ref, (budget, got[-1], ref)
