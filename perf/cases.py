"""The calls whose speed counts, with sizes, inputs, work and tolerances.

Each case is one call (or the calls a program makes together) of the blocked
SGD library through its Python binding: the epoch sweep in its placements,
the RMSE pass, held-out RMSE, loading (bucketing) ratings, and the outer
loop.  Sizes are those of the benchmark workloads in workloads/synth.py (the
two largest, 250M and 2e9 ratings, with fewer ratings on the same matrix, so
that inputs are quick to draw) and of the random-configuration tests.

Inputs are drawn on the GPU from the seed: distinct cells, heavy-tailed
degrees (users lognormal or Zipf, items Zipf, both saturating at the matrix's
edge), a planted low-rank model with noise, and a random order.
"""
import math

import numpy as np
import torch

from paper_2304_13724_amd import bgmf


def listed():
    return [
        # first use of the method, and the smallest epoch: uniform cells, few
        # row-blocks (the "tiny" workload)
        dict(name="epoch_tiny", kind="epoch", n=2_000, m=1_000, nnz=100_000, k=16, p=4,
             users="uniform", items=0.0, values="int5", rank=8, alpha=0.01, beta=0.05,
             blocks="equal"),
        # the paper's Table 1: a dense matrix of integers in 1..30
        dict(name="epoch_dense", kind="epoch", n=1_024, m=1_024, nnz=1_048_576, k=16, p=32,
             users="dense", items=0.0, values="uint", rank=0, alpha=2e-4, beta=5e-3,
             blocks="equal"),
        # odd sizes: blocks of unequal width, k not a power of two
        dict(name="epoch_ragged", kind="epoch", n=20_011, m=7_001, nnz=1_000_003, k=80, p=61,
             users="zipf0.8", items=0.9, values="int5", rank=16, alpha=0.005, beta=0.05,
             blocks="equal"),
        # ten million ratings (the "medium" workload)
        dict(name="epoch_medium", kind="epoch", n=70_000, m=10_000, nnz=10_000_000, k=32, p=256,
             users="zipf1.0", items=1.1, values="int5", rank=16, alpha=0.01, beta=0.05,
             blocks="equal"),
        # the headline workload: a hundred million ratings, the paper's equal blocks
        dict(name="epoch_large", kind="epoch", n=480_000, m=18_000, nnz=100_000_000, k=64, p=1024,
             users="lognormal1.2116", items=1.2, values="int5", rank=32, alpha=0.005, beta=0.05,
             blocks="equal"),
        # the same with cut points that balance the ratings over the blocks
        dict(name="epoch_large_balanced", kind="epoch", n=480_000, m=18_000, nnz=100_000_000,
             k=64, p=1024, users="lognormal1.2116", items=1.2, values="int5", rank=32,
             alpha=0.005, beta=0.05, blocks="balanced"),
        # the 250M-rating workload's matrix (k = 128, column slices too wide
        # for LDS, V in global memory)
        dict(name="epoch_wide", kind="epoch", n=1_000_000, m=625_000, nnz=100_000_000, k=128,
             p=2048, users="zipf1.1", items=1.1, values="cont100", rank=16, alpha=5e-4, beta=0.02,
             blocks="equal"),
        # the 2e9-rating workload's matrix, ratings streamed from host memory
        # under a device budget of half their size
        dict(name="epoch_streamed", kind="epoch", n=10_000_000, m=5_000_000, nnz=20_000_000, k=64,
             p=4096, users="zipf1.1", items=1.1, values="int5", rank=16, alpha=0.005, beta=0.05,
             blocks="streamed"),
        # the RMSE pass that follows every epoch of the headline workload
        dict(name="rmse_large", kind="rmse", n=480_000, m=18_000, nnz=100_000_000, k=64, p=1024,
             users="lognormal1.2116", items=1.2, values="int5", rank=32, alpha=0.005, beta=0.05,
             blocks="equal"),
        # test RMSE: ten million held-out ratings in device memory, no order
        dict(name="rmse_heldout", kind="heldout", n=480_000, m=18_000, nnz=10_000_000, k=64,
             p=1024, users="lognormal1.2116", items=1.2, values="int5", rank=32, alpha=0.005,
             beta=0.05, blocks="equal"),
        # loading ten million ratings from host arrays, and reading the layout
        dict(name="load_medium", kind="load", n=70_000, m=10_000, nnz=10_000_000, k=32, p=256,
             users="zipf1.0", items=1.1, values="int5", rank=16, alpha=0.01, beta=0.05,
             blocks="equal"),
        # Algorithm 1's outer loop on a small matrix: five epochs, each with
        # its RMSE pass
        dict(name="fit_tiny", kind="fit", n=2_000, m=1_000, nnz=100_000, k=16, p=4,
             users="uniform", items=0.0, values="int5", rank=8, alpha=0.01, beta=0.05,
             blocks="equal"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same kinds: matrices from 500 x 300 to 1M x 600K, fifty
    thousand to thirty million ratings, 60 to 6,000 ratings per block on
    average, every width k the library takes."""
    kind = rng.choice(["epoch", "epoch", "epoch", "epoch", "rmse", "heldout", "load", "fit"])
    nnz = _log(rng, 50_000, 1_000_000 if kind == "fit" else 30_000_000)
    users = rng.choice(["uniform", "zipf0.8", "zipf1.0", "zipf1.1", "lognormal1.0",
                        "lognormal1.2116"])
    per_row = _log(rng, 20, 400)
    n = min(max(nnz // per_row, 500), 1_000_000)
    m = min(max(int(n * math.exp(rng.uniform(math.log(0.03), math.log(0.8)))), 300), 600_000)
    while n * m < 5 * nnz:
        n, m = n + n // 2 + 1, m + m // 2 + 1
    p = int(round(math.sqrt(nnz / _log(rng, 60, 6_000))))
    p = max(2, min(p, n, m, 4096))
    while m > p * 60_000 or n > p * 60_000:
        p += 1
    k = rng.choice([16, 32, 48, 64, 64, 80, 128, 128, 256])
    if kind == "epoch":
        blocks = rng.choice(["equal", "equal", "equal", "balanced", "streamed"])
    else:
        blocks = "equal"
    if blocks == "streamed":
        p = max(p, 16)
    return dict(kind=kind, n=n, m=m, nnz=nnz, k=k, p=p, users=users,
                items=0.0 if users == "uniform" else rng.choice([0.9, 1.1, 1.2]),
                values="int5", rank=16, alpha=0.005, beta=0.05, blocks=blocks)


# ------------------------------------------------------------------ inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _degrees(g, n, m, total, spec):
    """Expected ratings per user, between 1 and m, summing to about total."""
    dev = g.device
    if spec.startswith("zipf"):
        raw = torch.arange(1, n + 1, device=dev, dtype=torch.float64) ** -float(spec[4:])
        raw = raw[torch.randperm(n, generator=g, device=dev)]
    else:
        z = torch.randn(n, generator=g, device=dev, dtype=torch.float64)
        raw = torch.exp(float(spec[9:]) * z)
    scale = total / raw.sum()
    for _ in range(40):
        d = (raw * scale).clamp(1.0, float(m))
        free = (raw * scale < m) & (raw * scale > 1.0)
        room = (raw * scale)[free].sum()
        if room <= 0:
            break
        scale = scale * (1.0 + (total - d.sum()) / room).clamp(0.2, 5.0)
    return (raw * scale).clamp(1.0, float(m))


def _bernoulli(g, lam, w, row_ids, col0, m):
    """Keys row * m + rank of the cells (row_ids x ranks col0..) drawn with
    probability 1 - exp(-lam w) each."""
    out = []
    step = max(1, (1 << 26) // max(1, w.numel()))
    for a in range(0, lam.numel(), step):
        pr = -torch.expm1(-lam[a:a + step, None].float() * w[None, :].float())
        hit = torch.rand(pr.shape, generator=g, device=g.device) < pr
        r, c = hit.nonzero(as_tuple=True)
        out.append(row_ids[a:a + step][r] * m + (c + col0))
    return out


def _cells(g, n, m, nnz, users, items):
    """Keys row * m + column of nnz distinct cells, in random order."""
    dev = g.device
    if users == "dense":
        return torch.randperm(n * m, generator=g, device=dev)[:nnz]
    if users == "uniform":
        want = int(nnz * (1.02 + nnz / (n * m)) + 1000)
        key = torch.empty(0, dtype=torch.int64, device=dev)
        while key.numel() < nnz:
            more = torch.randint(0, n * m, (want,), generator=g, device=dev)
            key = torch.unique(torch.cat([key, more]))
    else:
        # user i rates item j with probability 1 - exp(-lam_i w_j): sampling
        # without replacement by Zipf item weights, lam_i set by the degree
        w = torch.arange(1, m + 1, device=dev, dtype=torch.float64) ** -items
        w /= w.sum()
        d = _degrees(g, n, m, nnz * 1.01, users)
        grid = torch.logspace(-1, 9, 161, device=dev, dtype=torch.float64)
        dist = torch.stack([-torch.expm1(-x * w).sum() for x in grid])
        at = torch.searchsorted(dist, d).clamp(1, grid.numel() - 1)
        lo, hi = dist[at - 1], dist[at]
        f = ((d - lo) / (hi - lo).clamp_min(1e-9)).clamp(0, 1)
        lam = grid[at - 1] * (grid[at] / grid[at - 1]) ** f
        heavy = d > m / 8
        ids = torch.arange(n, device=dev)
        parts = _bernoulli(g, lam[heavy], w, ids[heavy], 0, m)
        lam, ids = lam[~heavy], ids[~heavy]
        head = min(m, max(16, min(512, int(4e8 // n))))
        parts += _bernoulli(g, lam, w[:head], ids, 0, m)
        if head < m:
            count = torch.poisson(lam * w[head:].sum(), generator=g).to(torch.int64)
            cdf = torch.cumsum(w[head:], 0)
            cdf /= cdf[-1].clone()
            tail = []
            ends = torch.cumsum(count, 0)
            a = 0
            while a < ids.numel():  # about 2^26 draws at a time
                base = int(ends[a - 1]) if a else 0
                b = int(torch.searchsorted(ends, torch.tensor(base + (1 << 26), device=dev)))
                b = max(a + 1, min(b, ids.numel()))
                r = torch.repeat_interleave(ids[a:b], count[a:b])
                x = torch.rand(r.numel(), generator=g, device=dev, dtype=torch.float64)
                c = torch.searchsorted(cdf, x).clamp_max(m - head - 1) + head
                tail.append(torch.unique(r * m + c))
                a = b
            parts += tail
        key = torch.cat(parts)
        del parts
        item = torch.randperm(m, generator=g, device=dev)
        key = (key // m) * m + item[key % m]
    return key[torch.randperm(key.numel(), generator=g, device=dev)[:nnz]]


def _ratings(case, seed):
    """rows, cols (int32) and vals (float32) of the case, on the device."""
    n, m = case["n"], case["m"]
    g = torch.Generator(device=_device())
    g.manual_seed(seed)
    key = _cells(g, n, m, case["nnz"], case["users"], case["items"])
    rows, cols = (key // m).to(torch.int32), (key % m).to(torch.int32)
    del key
    count = rows.numel()
    if case["values"] == "uint":
        vals = torch.randint(1, 31, (count,), generator=g, device=g.device).float()
        return rows, cols, vals
    rank = case["rank"]
    us = torch.randn(n, rank, generator=g, device=g.device) / rank ** 0.5
    vs = torch.randn(m, rank, generator=g, device=g.device) / rank ** 0.5
    z = torch.empty(count, device=g.device)
    for a in range(0, count, 1 << 24):
        r, c = rows[a:a + (1 << 24)].long(), cols[a:a + (1 << 24)].long()
        z[a:a + (1 << 24)] = (us[r] * vs[c]).sum(1)
    if case["values"] == "int5":
        z += 3.0 - z.mean() + 0.5 * torch.randn(count, generator=g, device=g.device)
        vals = z.round_().clamp_(1.0, 5.0)
    else:
        z = 50.0 + 20.0 * (z - z.mean()) / z.std().clamp_min(1e-6)
        z += 5.0 * torch.randn(count, generator=g, device=g.device)
        vals = z.clamp_(0.0, 100.0)
    return rows, cols, vals


def _factors(case, seed):
    g = torch.Generator(device=_device())
    g.manual_seed(seed + 77_777)
    U = torch.rand(case["n"], case["k"], generator=g, device=g.device) * 0.1
    V = torch.rand(case["m"], case["k"], generator=g, device=g.device) * 0.1
    if case["kind"] in ("rmse", "heldout"):
        # trained factors: products spread around the mean rating
        U += 0.3 * torch.randn(case["n"], case["k"], generator=g, device=g.device) / case["k"] ** 0.5
        V += (3.0 / (0.05 * case["k"])) * (0.9 + 0.2 * torch.rand(
            case["m"], case["k"], generator=g, device=g.device))
    return U, V


def prepare(case, seed):
    rows, cols, vals = _ratings(case, seed)
    n, m, k, p = case["n"], case["m"], case["k"], case["p"]
    mdl = bgmf.Model(n, m, k, p)
    st = dict(case=case, mdl=mdl)
    if case["kind"] == "load":
        st["coo"] = tuple(a.cpu().numpy() for a in (rows, cols, vals))
        return st
    # torch's allocator owns every buffer, as in a program built on torch
    U, V = _factors(case, seed)
    sizes = mdl.query_sizes(rows.numel())
    if case["kind"] == "heldout":
        ws = torch.empty(sizes["min_ws_bytes"], dtype=torch.uint8, device=U.device)
        mdl.bind_tensors(U, V, ws)
        st.update(U=U, V=V, ws=ws, dev=(rows, cols, vals))
        torch.cuda.synchronize()
        return st
    host = tuple(a.cpu().numpy() for a in (rows, cols, vals))
    count = rows.numel()
    del rows, cols, vals
    if case["blocks"] == "balanced":
        mdl.set_cuts(*bgmf.bgmf_balanced_cuts(n, m, p, host[0], host[1], max_cols=max(
            64, -(-m // p))))
    pinned = None
    if case["blocks"] == "streamed":
        pinned = torch.empty(sizes["pinned_bytes"], dtype=torch.uint8, pin_memory=True)
        mdl.set_option(bgmf.BGMF_OPT_RATINGS_BUDGET, max(4 * count, 1 << 20))
    ws = torch.empty(sizes["incore_ws_bytes"], dtype=torch.uint8, device=U.device)
    torch.cuda.synchronize()
    mdl.bind_tensors(U, V, ws, pinned)
    mdl.load_coo(*host)
    st.update(U=U, V=V, ws=ws, pinned=pinned)
    return st


# ------------------------------------------------------------------ one pass

_FIT_EPOCHS = 5


def run(st):
    case, mdl = st["case"], st["mdl"]
    kind = case["kind"]
    if kind == "epoch":
        mdl.epoch(case["alpha"], case["beta"])
        return {"U": st["U"], "V": st["V"]}
    if kind == "fit":
        ran, hist = mdl.fit(case["alpha"], case["beta"], _FIT_EPOCHS, 0.0)
        return {"epochs": ran, "rmse": hist, "U": st["U"], "V": st["V"]}
    if kind == "rmse":
        return mdl.rmse()
    if kind == "heldout":
        rows, cols, vals = st["dev"]
        return bgmf.bgmf_rmse_coo_dev(mdl.h, rows.data_ptr(), cols.data_ptr(), vals.data_ptr(),
                                      rows.numel())
    mdl.load_coo(*st["coo"])
    block_ptr, perm = mdl.get_layout()
    return {"block_ptr": block_ptr, "perm": perm}


def work(case):
    """Bytes: the ratings (12 bytes each) read once, U and V read and, where
    they are updated, written once, other outputs written once.  Operations:
    2k per dot product, 4k per updated vector."""
    n, m, k, p, nnz = (case[x] for x in ("n", "m", "k", "p", "nnz"))
    factors = 4 * k * (n + m)
    kind = case["kind"]
    if kind == "load":
        return {"bytes": 12 * nnz + 8 * nnz + 4 * nnz + 8 * (p * p + 1), "flops": 0}
    if kind in ("rmse", "heldout"):
        return {"bytes": 12 * nnz + factors, "flops": (2 * k + 3) * nnz}
    epoch = {"bytes": 12 * nnz + 2 * factors, "flops": 10 * k * nnz}
    if kind == "epoch":
        return epoch
    return {"bytes": _FIT_EPOCHS * epoch["bytes"] + (_FIT_EPOCHS + 1) * (12 * nnz + factors),
            "flops": _FIT_EPOCHS * epoch["flops"] + (_FIT_EPOCHS + 1) * (2 * k + 3) * nnz}


def tolerance(case):
    kind = case["kind"]
    if kind == "load":
        return "exact"
    if kind in ("rmse", "heldout"):
        return {"rel": 5e-7}
    # about four times the distance of an epoch in 32 bits from one in 64
    # (U and V at most 9e-7, largest difference 2.4e-5; ratings in [0, 100]
    # with k = 128 amplify it over the epoch: 4.6e-5 and 3.3e-3)
    if case["values"] == "cont100":
        return {"rel": 2e-4, "max": 1.3e-2}
    return {"rel": 4e-6, "max": 1e-4}


# ------------------------------------------------------------------ in 64 bits

# numpy steps a reference may take (one step: the t-th ratings of all blocks
# of a stratum), about 15 seconds
_EXACT_STEPS = 160_000


def _exact_rmse(rows, cols, vals, U, V):
    total = torch.zeros((), dtype=torch.float64, device=vals.device)
    for a in range(0, vals.numel(), 1 << 21):
        r, c = rows[a:a + (1 << 21)].long(), cols[a:a + (1 << 21)].long()
        d = vals[a:a + (1 << 21)].double() - (U[r].double() * V[c].double()).sum(1)
        total += (d * d).sum()
    return math.sqrt(float(total) / vals.numel())


def _exact_epoch(case, rows, cols, vals, U, V, cuts, passes_done):
    """One epoch on float64 arrays U and V, in place; False if too long."""
    n, m, p = case["n"], case["m"], case["p"]
    rc, cc = cuts
    R = np.searchsorted(rc, rows, side="right") - 1
    C = np.searchsorted(cc, cols, side="right") - 1
    slot = ((C - R) % p) * p + R
    order = np.lexsort((np.arange(rows.size), rows, slot))
    start = np.searchsorted(slot[order], np.arange(p * p + 1)).reshape(-1)
    lens = np.diff(start).reshape(p, p)
    if lens.max(axis=1).sum() * passes_done > _EXACT_STEPS:
        return False
    a, b = float(np.float32(case["alpha"])), float(np.float32(case["beta"]))
    for s in range(p):
        by_len = np.argsort(-lens[s], kind="stable")
        ln = lens[s][by_len]
        first = start[s * p + by_len]
        for t in range(int(ln[0]) if ln.size else 0):
            live = int(np.searchsorted(-ln, -t, side="left"))  # blocks longer than t
            e = order[first[:live] + t]
            i, j = rows[e], cols[e]
            u, v = U[i], V[j]
            err = a * (vals[e] - np.einsum("ij,ij->i", u, v))[:, None]
            U[i] = u + err * v - (a * b) * u
            V[j] = v + err * u - (a * b) * v
    return True


def exact(case, seed):
    kind = case["kind"]
    if kind == "load" or case["nnz"] * case["k"] > 6_400_000_000:
        return None
    rows, cols, vals = _ratings(case, seed)
    U, V = _factors(case, seed)
    if kind in ("rmse", "heldout"):
        return _exact_rmse(rows, cols, vals, U, V)
    if case["blocks"] == "balanced" or case["nnz"] > 12_000_000:
        return None
    n, m, p = case["n"], case["m"], case["p"]
    cuts = [-(-np.arange(p + 1) * x // p) for x in (n, m)]
    epochs = _FIT_EPOCHS if kind == "fit" else 1
    r, c, x = rows.cpu().numpy(), cols.cpu().numpy(), vals.cpu().numpy().astype(np.float64)
    Ud, Vd = U.cpu().numpy().astype(np.float64), V.cpu().numpy().astype(np.float64)

    def rmse():
        return _exact_rmse(rows, cols, vals, torch.from_numpy(Ud).to(vals.device),
                           torch.from_numpy(Vd).to(vals.device))

    hist = [rmse()] if kind == "fit" else None
    for _ in range(epochs):
        if not _exact_epoch(case, r, c, x, Ud, Vd, cuts, epochs):
            return None
        if kind == "fit":
            hist.append(rmse())
    if kind == "epoch":
        return {"U": Ud, "V": Vd}
    return {"epochs": None, "rmse": np.array(hist), "U": Ud, "V": Vd}
