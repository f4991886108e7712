"""Timed cases of the library: what its users have it do, called the way their programs call it.

A case is one call (or one short series of calls) through the binding `paper_2202_09512_amd`: a fit of a perturbed
ensemble at a fixed rank from given starting factors, one iteration without a handle, a fit with threshold checks, or a
whole rank selection; on dense, sparse, power-law and binary tensors.  `exact` states the same results in plain torch in
64 bits.  Inputs are drawn on the GPU from the seed.
"""
import itertools
import math

import numpy as np
import torch

import paper_2202_09512_amd as nn

DELTA, EPS = 0.03, 1e-16      # perturbation half-width and division guard of the paper's experiments


# ------------------------------------------------------------------------------------------------- the cases
def _case(kind, data, n, m, k, q, iters, **more):
    c = dict(kind=kind, data=data, n=n, m=m, k=k, q=q, iters=iters, entries=0, deterministic=False, k_lo=0)
    c.update(more)
    return c


def listed():
    return [
        # one iteration of a caller that may not allocate (a serving loop, code under capture): all latency
        dict(_case("static", "dense", 100, 3, 5, 4, 1), name="static_100"),
        # the small end of the synthetic sweep: 64 entities, 4 relations, 200 iterations of every member
        dict(_case("fit", "dense", 64, 4, 3, 10, 200), name="tiny_64"),
        # a few hundred entities, an odd size: a handful of small kernels per iteration
        dict(_case("fit", "dense", 333, 5, 8, 10, 20), name="small_333"),
        # the demonstration tensor of 1024 x 1024 x 10, with the stopping rule looked at every fifth iteration
        dict(_case("until", "dense", 1024, 10, 10, 10, 10), name="until_1024"),
        # dense medium: 20 members at the top rank of the sweep 2..16 (two whole groups of 8 and a tail of 4)
        dict(_case("fit", "dense", 2048, 16, 16, 20, 4), name="medium_2048"),
        # the larger demonstration tensor, 2160 x 2160 x 20, above the planted rank: two 16-column blocks
        dict(_case("fit", "dense", 2160, 20, 24, 10, 2), name="wide_2160"),
        # dense large: 34 GB, one ensemble iteration
        dict(_case("fit", "dense", 16384, 32, 16, 8, 1), name="large_16384"),
        # the reproducible mode on an odd size (rows that are not 16-byte aligned)
        dict(_case("fit", "dense", 1501, 6, 12, 6, 5, deterministic=True), name="repro_1501"),
        # sparse: a million entities in communities, 8e7 stored entries, given as CSR
        dict(_case("fit", "community", 1_000_000, 8, 32, 4, 2, entries=10_000_000), name="sparse_1e6"),
        # sparse with power-law rows and columns at the highest rank
        dict(_case("fit", "powerlaw", 2_000_000, 4, 64, 2, 2, entries=10_000_000), name="powerlaw_2e6"),
        # a knowledge graph: binary triples over 24 relations, most entities without an entry in most relations
        dict(_case("fit", "triples", 20_000, 24, 16, 8, 10, entries=25_000), name="triples_20000"),
        # the method as a whole: fits, clustering, silhouettes, regression and the choice of the rank
        dict(_case("select", "dense", 500, 6, 6, 8, 40, k_lo=2), name="select_500"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["static", "tiny", "dense", "dense", "dense", "until", "repro", "community", "powerlaw", "triples", "select"])
    if kind == "static":
        return _case("static", "dense", rng.randint(20, 400), rng.randint(1, 6), rng.randint(2, 16), rng.randint(1, 12), 1)
    if kind == "tiny":
        return _case("fit", "dense", rng.randint(16, 64), rng.randint(1, 6), rng.randint(2, 6), rng.randint(2, 20),
                     rng.randint(50, 200))
    if kind in ("dense", "until", "repro"):
        n = _log(rng, 130, 8000)
        m = max(1, min(rng.randint(1, 24), int(6e8 / n ** 2)))
        k = rng.choice([rng.randint(2, 16), rng.randint(2, 16), rng.randint(17, 32), rng.randint(33, 64)])
        q = rng.randint(1, 24)
        one = m * n * n * q * max(1, -(-k // 16))        # the largest listed case makes 6.9e10
        if one > 3e10:
            q = max(1, int(q * 3e10 / one))
            one = m * n * n * q * max(1, -(-k // 16))
        iters = max(1, min(10, int(3e10 / one)))
        if kind == "until":
            return _case("until", "dense", n, m, k, q, max(2, iters))
        return _case("fit", "dense", n, m, k, q, iters, deterministic=kind == "repro")
    if kind == "community":
        n = _log(rng, 20_000, 1_000_000)
        return _case("fit", "community", n, rng.randint(2, 8), rng.randint(2, 48), rng.randint(1, 5), 2,
                     entries=int(n * rng.uniform(2, 9)), deterministic=rng.random() < 0.25)
    if kind == "powerlaw":
        n = _log(rng, 50_000, 2_000_000)
        return _case("fit", "powerlaw", n, rng.randint(1, 4), rng.randint(8, 64), rng.randint(1, 2), 2,
                     entries=int(n * rng.uniform(1, 5)))
    if kind == "triples":
        n = _log(rng, 2_000, 40_000)
        return _case("fit", "triples", n, rng.randint(4, 40), rng.randint(4, 24), rng.randint(2, 10), rng.randint(3, 10),
                     entries=int(n * rng.uniform(0.3, 4)))
    k_hi = rng.randint(4, 7)
    return _case("select", "dense", _log(rng, 100, 900), rng.randint(2, 6), k_hi, rng.randint(3, 10), 40, k_lo=max(2, k_hi - 4))


# ------------------------------------------------------------------------------------------------- inputs
def _planted_factors(n, m, rank, g, dev):
    """Communities: every entity has one dominant column, the others are small; cores uniform."""
    A = 0.05 * torch.rand((n, rank), generator=g, device=dev)
    own = torch.arange(n, device=dev) * rank // n
    A[torch.arange(n, device=dev), own] = 0.5 + 0.5 * torch.rand(n, generator=g, device=dev)
    return A, torch.rand((m, rank, rank), generator=g, device=dev)


def _dense_tensor(c, g, dev):
    n, m = c["n"], c["m"]
    rank = 16 if n >= 8192 else (c["k"] if c["kind"] != "select" else max(2, c["k"] - 2))
    rank = min(rank, 16, n)
    A, R = _planted_factors(n, m, rank, g, dev)
    X = torch.empty((m, n, n), device=dev)
    for t in range(m):
        x = (A @ R[t]) @ A.T
        x *= 1.0 + 0.01 * torch.randn((n, n), generator=g, device=dev)
        X[t] = x.clamp_(min=0.0)
    return X


def _positions(c, g, dev, ids, cdf):
    """Sorted, distinct positions row * n + column of one relation."""
    n, cnt = c["n"], c["entries"]
    ri = lambda hi, k: torch.randint(0, hi, (k,), generator=g, device=dev)
    if c["data"] == "community":                      # 90 % inside one of 32 diagonal blocks of entities
        size, inside = n // 32, int(0.9 * cnt)
        block = ri(32, inside) * size
        rows = torch.cat([block + ri(size, inside), ri(n, cnt - inside)])
        cols = torch.cat([block + ri(size, inside), ri(n, cnt - inside)])
    else:                                             # Zipf(1.1) over permuted entity ids
        u = lambda: torch.rand(cnt, generator=g, device=dev, dtype=torch.float64)
        rows = ids[torch.searchsorted(cdf, u()).clamp_(max=n - 1)]
        cols = ids[torch.searchsorted(cdf, u()).clamp_(max=n - 1)]
    return torch.unique(rows * n + cols)


def _sparse_tensor(c, g, dev):
    """(row pointers [m][n+1], columns, values or None, offsets of the slices): CSR per relation."""
    n, m = c["n"], c["m"]
    A, R = _planted_factors(n, m, 32, g, dev)
    ids = cdf = None
    if c["data"] != "community":
        ids = torch.randperm(n, generator=g, device=dev)
        cdf = torch.cumsum(torch.arange(1, n + 1, dtype=torch.float64, device=dev) ** -1.1, 0)
        cdf /= cdf[-1].clone()
    ptr = torch.zeros((m, n + 1), dtype=torch.int64, device=dev)
    cols, vals, off = [], [], [0]
    for t in range(m):
        key = _positions(c, g, dev, ids, cdf)
        i, j = key // n, key % n
        ptr[t, 1:] = torch.cumsum(torch.bincount(i, minlength=n), 0)
        cols.append(j.to(torch.int32))
        if c["data"] != "triples":
            v = ((A[i] @ R[t]) * A[j]).sum(1)
            if c["data"] == "powerlaw":
                v *= 1.0 - torch.rand(v.numel(), generator=g, device=dev)
            vals.append(v)
        off.append(off[-1] + key.numel())
    return ptr, torch.cat(cols), torch.cat(vals) if vals else None, off


def _inputs(c, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    X = _dense_tensor(c, g, dev) if c["data"] == "dense" else _sparse_tensor(c, g, dev)
    # the starting factors: uniform in (0, 1), as the method's random start
    A0 = torch.rand((c["q"], c["n"], c["k"]), generator=g, device=dev) + 2.0 ** -24
    R0 = torch.rand((c["q"], c["m"], c["k"], c["k"]), generator=g, device=dev) + 2.0 ** -24
    return X, A0, R0


def prepare(case, seed):
    c = case
    X, A0, R0 = _inputs(c, seed)
    T = nn.DenseX(X) if c["data"] == "dense" else nn.SparseX(c["n"], c["m"], *X)
    h = None
    if c["kind"] in ("fit", "until"):
        h = _Fit(nn.nnrescal_init(T, k=c["k"], q=c["q"], delta=DELTA, eps_div=EPS, seed=seed, A0=A0, R0=R0,
                                  deterministic=c["deterministic"]))
    return dict(case=c, seed=seed, X=X, T=T, A0=A0, R0=R0, fit=h)


class _Fit:
    """A fit's handle, released with the program's last reference to it."""

    def __init__(self, h):
        self.h = h

    def __del__(self):
        nn.nnrescal_destroy(self.h)


def _padded(a, shape):
    """The chosen rank's factors in arrays of the largest rank's shape: which rank is chosen depends on the inputs."""
    out = torch.zeros(shape, dtype=a.dtype, device=a.device)
    out[tuple(slice(0, d) for d in a.shape)] = a
    return out


def run(state):
    c, T = state["case"], state["T"]
    if c["kind"] == "static":
        A, R = state["A0"].clone(), state["R0"].clone()
        nn.nnrescal_mu_step_static(T, A, R, delta=DELTA, eps_div=EPS, seed=state["seed"])
        return {"A": A, "R": R}
    if c["kind"] == "select":
        s = nn.nnrescal_select_k(T, c["k_lo"], c["k"], q=c["q"], delta=DELTA, iters=c["iters"], seed=state["seed"], eps_div=EPS,
                                 regress_iters=100)
        return {"s_min": np.array(s["s_min"], np.float32), "s_avg": np.array(s["s_avg"], np.float32),
                "err": np.array(s["err"], np.float32), "A": _padded(s["A_med"], (c["n"], c["k"])),
                "R": _padded(s["R_reg"], (c["m"], c["k"], c["k"]))}
    h = state["fit"].h
    nn.nnrescal_set_factors(h, state["A0"], state["R0"])
    out = {}
    if c["kind"] == "until":                          # a threshold that is never met: checks, and all iterations
        done, trace = nn.nnrescal_fit_until(h, c["iters"], 0.0, check_every=max(1, c["iters"] // 2))
        out = {"done": done, "trace": np.array(trace, np.float64)}
    else:
        nn.nnrescal_fit(h, c["iters"])
    out["A"], out["R"] = nn.nnrescal_get_factors(h)
    return out


# ------------------------------------------------------------------------------------------------- floors
def work(case):
    c = case
    n, m, q = c["n"], c["m"], c["q"]

    def iteration(k):
        pairs = m * n * n if c["data"] == "dense" else m * c["entries"]
        # X_t A and X_t^T A; A^T A and A W; A^T (X_t A); (X_t A) R_t^T and (X_t^T A) R_t; six k x k products per slice
        return q * (4.0 * pairs * k + 4.0 * n * k * k + 6.0 * m * n * k * k + 12.0 * m * k ** 3)

    if c["data"] == "dense":
        x = 4.0 * m * n * n
    else:
        x = (4.0 if c["data"] == "triples" else 8.0) * m * c["entries"] + 8.0 * m * n
    factors = lambda k: 8.0 * q * (n * k + m * k * k)   # read and written
    ks = range(c["k_lo"], c["k"] + 1) if c["kind"] == "select" else [c["k"]]
    # a tensor that the caches hold (256 MB) need not be read again by the next iteration, nor by the next rank
    times = c["iters"] * len(ks) if x > 256e6 else 1
    return {"bytes": x * times + sum(factors(k) for k in ks), "flops": c["iters"] * sum(iteration(k) for k in ks)}


def tolerance(case):
    # measured against 64 bits: up to 1.6e-6 on factors, objective and silhouettes (200 iterations of sums in 32 bits, finished
    # in any order); the sweep's silhouettes and cores also pass through the starts' worst member
    return {"rel": 3e-5, "max": 3e-4} if case["kind"] == "select" else {"rel": 8e-6, "max": 1e-4}


# ------------------------------------------------------------------------------------------------- 64 bits
def _philox(e, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) of the counters (e, c2, c3): four tensors of 32-bit words in int64."""
    low = 0xFFFFFFFF
    signed = lambda v: v - (1 << 64) if v >= 1 << 63 else v
    c0, c1 = e & low, (e >> 32) & low
    c2, c3 = torch.full_like(e, c2), torch.full_like(e, c3)
    k0, k1 = seed & low, (seed >> 32) & low
    for _ in range(10):
        p0, p1 = c0 * signed(0xD2511F53), c2 * signed(0xCD9E8D57)       # modulo 2^64
        c0, c2 = ((p1 >> 32) & low) ^ c1 ^ k0, ((p0 >> 32) & low) ^ c3 ^ k1
        c1, c3 = p1 & low, p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return c0, c1, c2, c3


def _perturbed(x, e, t, group, seed, members):
    """The values x (float32, at coordinates e = i n + j of slice t) as the given members of a group of 8 see them: with h
    the member's 16-bit draw, fl(fl(x a) h + fl(x c)), a = 2 d, c = fl(1 - 65535 d), d = fl(delta 2^-16)."""
    d = torch.tensor(DELTA, dtype=torch.float32, device=x.device) * 2.0 ** -16
    cc = (1.0 - 65535.0 * d.double()).float()
    xa, xc = (x * (2.0 * d)).double(), (x * cc).double()
    w = _philox(e, t, group, seed)
    for r in members:
        h = (w[r >> 1] >> (16 * (r & 1))) & 0xFFFF
        yield r, (xa * h + xc).float()                # (exact in 64 bits before the one rounding)


def _products(c, X, A, seed, kept=None):
    """P[t], Q[t] = X^r_t A^r, X^r_t^T A^r for all members: lists over t of [q][n][k] float64.  kept: a dict that holds the
    perturbed values between the iterations of one fit."""
    n, m, q = c["n"], c["m"], c["q"]
    dev = A.device
    P = [torch.empty_like(A) for _ in range(m)]
    Q = [torch.empty_like(A) for _ in range(m)]
    for t in range(m):
        for grp in range((q + 7) // 8):
            members = range(min(8, q - 8 * grp))
            if c["data"] == "dense":
                rows = max(1, (1 << 26) // n)
                for i0 in range(0, n, rows):
                    x = X[t, i0:i0 + rows]
                    if kept is None or (t, grp, i0) not in kept:
                        e = (torch.arange(i0, i0 + x.shape[0], device=dev) * n)[:, None] + torch.arange(n, device=dev)
                        got = list(_perturbed(x, e, t, grp, seed, members))
                        if kept is not None:
                            kept[t, grp, i0] = got
                    else:
                        got = kept[t, grp, i0]
                    for r, xq in got:
                        xq, a = xq.double(), A[8 * grp + r]
                        P[t][8 * grp + r, i0:i0 + rows] = xq @ a
                        part = xq.T @ a[i0:i0 + rows]
                        if i0 == 0:
                            Q[t][8 * grp + r] = part
                        else:
                            Q[t][8 * grp + r] += part
                continue
            ptr, cols, vals, off = X
            lens = ptr[t, 1:] - ptr[t, :-1]
            i = torch.repeat_interleave(torch.arange(n, device=dev), lens)
            j = cols[off[t]:off[t + 1]].long()
            v = torch.ones(j.numel(), device=dev) if vals is None else vals[off[t]:off[t + 1]]
            order = torch.argsort(j * n + i)
            jlens = torch.bincount(j, minlength=n)
            for r, xq in _perturbed(v, i * n + j, t, grp, seed, members):
                xq, a = xq.double()[:, None], A[8 * grp + r]
                P[t][8 * grp + r] = _segment_sums(lambda s: xq[s] * a[j[s]], lens, a.shape[1])
                Q[t][8 * grp + r] = _segment_sums(lambda s: xq[order[s]] * a[i[order[s]]], jlens, a.shape[1])
    return P, Q


def _segment_sums(term, lens, k):
    """Sums of neighbouring rows of term(slice), lens[i] of them for row i; a bounded number of rows at a time."""
    out = torch.zeros((lens.numel(), k), dtype=torch.float64, device=lens.device)
    ends = torch.cumsum(lens, 0)
    step = max(1, (1 << 28) // k)
    total, lo, row = int(ends[-1]), 0, 0
    while lo < total:
        last = int(torch.searchsorted(ends, torch.tensor(min(total, lo + step), device=ends.device), right=True))
        last = max(last, row + 1)                     # rows [row, last)
        hi = int(ends[last - 1])
        if hi > lo:
            ids = torch.repeat_interleave(torch.arange(last - row, device=lens.device), lens[row:last])
            out[row:last].index_add_(0, ids, term(slice(lo, hi)))
        lo, row = hi, last
    return out


def _iterate(c, X, A, R, seed, iters, trace=None, check=0):
    """`iters` iterations of Eq. 2 (A [q][n][k], R [q][m][k][k], float64)."""
    kept = {} if c["data"] == "dense" and iters > 1 and 4.0 * c["q"] * c["m"] * c["n"] ** 2 < 6e10 else None
    for it in range(1, iters + 1):
        G = A.transpose(1, 2).contiguous() @ A
        P, Q = _products(c, X, A, seed, kept)
        num, W = torch.zeros_like(A), torch.zeros_like(G)
        At = A.transpose(1, 2).contiguous()
        look = trace is not None and it % check == 0
        f = torch.zeros(A.shape[0], dtype=torch.float64, device=A.device)
        Rn = torch.empty_like(R)
        for t in range(c["m"]):
            S, Rt = At @ P[t], R[:, t]
            GRG = G @ (Rt @ G)
            if look:
                f += (GRG * Rt).sum((1, 2)) - 2.0 * (S * Rt).sum((1, 2))
            Rt = Rt * S / (GRG + EPS)
            Rn[:, t] = Rt
            Rtt = Rt.transpose(1, 2).contiguous()
            num += P[t] @ Rtt + Q[t] @ Rt
            W += Rt @ (G @ Rtt) + Rtt @ (G @ Rt)
        if look:
            for grp in range((c["q"] + 7) // 8):
                members = range(min(8, c["q"] - 8 * grp))
                for t in range(c["m"]):
                    e = torch.arange(c["n"] ** 2, device=A.device).view(c["n"], c["n"])
                    for r, xq in _perturbed(X[t], e, t, grp, seed, members):
                        f[8 * grp + r] += xq.double().square().sum()
            trace.append(f)
        A, R = A * num / (A @ W + EPS), Rn
        del P, Q, num
    return A, R


def _unit(A, R):
    d = A.square().sum(1).sqrt()
    d = torch.where(d > 0, d, torch.ones_like(d))
    return A / d[:, None, :], R * d[:, None, :, None] * d[:, None, None, :]


def _start(c, k, seed, dev):
    """The method's random start: uniform draws keyed by the rank, the member and the element."""
    unit = lambda w: ((2 * (w >> 9) + 1).double() * 2.0 ** -24)
    A = torch.stack([unit(_philox(torch.arange(c["n"] * k, device=dev), k, (1 << 16) | r, seed)[0]).view(c["n"], k)
                     for r in range(c["q"])])
    R = torch.stack([unit(_philox(torch.arange(c["m"] * k * k, device=dev), k, (2 << 16) | r, seed)[0]).view(c["m"], k, k)
                     for r in range(c["q"])])
    return A, R


def _best_permutation(sim):
    k = sim.shape[0]
    perms = np.array(list(itertools.permutations(range(k))))
    return perms[np.argmax(sim[np.arange(k), perms].sum(1))]


def _cluster(A, R):
    """Alignment to a common order of the columns, medians, silhouettes on the cosine distance (normalised ensemble)."""
    q, n, k = A.shape
    A, R = A.cpu().numpy(), R.cpu().numpy()
    cols = A / np.linalg.norm(A, axis=1, keepdims=True)
    M, prev = A[0], None
    for _ in range(50):
        Mu = M / np.linalg.norm(M, axis=0)
        perm = np.array([_best_permutation(Mu.T @ cols[r]) for r in range(q)])
        M = np.median(np.stack([A[r][:, perm[r]] for r in range(q)]), axis=0)
        if prev is not None and (prev == perm).all():
            break
        prev = perm
    Rm = np.median(np.stack([R[r][:, perm[r]][:, :, perm[r]] for r in range(q)]), axis=0)
    pts = np.stack([cols[r][:, perm[r]].T for r in range(q)]).reshape(q * k, n)      # point (r, s)
    D = (1.0 - pts @ pts.T).reshape(q, k, q, k)
    sil = np.zeros((q, k))
    for r in range(q):
        for s in range(k):
            a = (D[r, s, :, s].sum() - D[r, s, r, s]) / (q - 1)
            b = min(D[r, s, :, u].mean() for u in range(k) if u != s)
            sil[r, s] = (b - a) / max(a, b) if max(a, b) else 0.0
    return M, Rm, sil.mean(0).min(), sil.mean()


def _select(c, X, seed):
    dev, X64 = X.device, X.double()
    res = []
    for k in range(c["k_lo"], c["k"] + 1):
        A, R = _start(c, k, seed, dev)
        A, R = _unit(*_iterate(c, X, A, R, seed, c["iters"]))
        M, Rm, smin, savg = _cluster(A, R)
        M, Rm = torch.from_numpy(M).to(dev), torch.from_numpy(np.maximum(Rm, 1e-12)).to(dev)
        Mt = M.T.contiguous()
        G, S = Mt @ M, torch.stack([Mt @ (x @ M) for x in X64])
        for _ in range(100):
            Rm = Rm * S / (torch.stack([G @ r @ G for r in Rm]) + EPS)
        err = math.sqrt(sum(float((x - M @ r @ Mt).square().sum()) for x, r in zip(X64, Rm)) / float(X64.square().sum()))
        res.append((smin, savg, err, M, Rm))
    score = [r[0] - r[2] for r in res]
    best = max(range(len(res)), key=lambda i: (score[i], i))
    return {"s_min": np.array([r[0] for r in res]), "s_avg": np.array([r[1] for r in res]),
            "err": np.array([r[2] for r in res]), "A": _padded(res[best][3], (c["n"], c["k"])),
            "R": _padded(res[best][4], (c["m"], c["k"], c["k"]))}


def exact(case, seed):
    c = case
    X, A0, R0 = _inputs(c, seed)
    if c["kind"] == "select":
        return _select(c, X, seed)
    trace = [] if c["kind"] == "until" else None
    A, R = _iterate(c, X, A0.double(), R0.double(), seed, c["iters"], trace, max(1, c["iters"] // 2))
    if trace is None:
        return {"A": A, "R": R}
    return {"done": c["iters"], "trace": np.array([f.cpu().numpy() for f in trace]), "A": A, "R": R}
