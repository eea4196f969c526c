"""Performance cases: the work a user has this library do, over the sizes it is used at.

Four paths, each through the public entry points of ``TuckerContext`` and
``TuckerEval``:

* ``hooi``    a decomposition: starting factors set, HOOI invocations run, the
              core, the fits and the factors read back;
* ``ttm``     the TTM-chain along every mode, for programs that run their own
              SVD step or optimiser on the penultimate matrices;
* ``fit``     one step of Tucker completion by gradient descent: the model at
              the observed coordinates, a loss, its gradients;
* ``ingest``  a new tensor: coordinates merged, ranks set (partition and
              layouts), factors set, and the first TTM-chains.

Tensors are drawn on the GPU: Zipf or uniform coordinates (exponent 0 is
uniform), lognormal values for ``ttm`` and ``ingest``.  The ``hooi`` tensors
hold a planted low-rank model plus noise at the drawn coordinates, and start
from factors that overlap the planted ones, as a run resumed from earlier
factors does; their spectra then separate the leading subspaces.
"""
import math

import numpy as np
import torch

import paper_1804_09494_amd as tk

DEV = "cuda:0"


def _case(name, path, dims, nnz, ranks, zipf=None, prec="fp32", iters=1):
    c = {"path": path, "dims": "x".join(map(str, dims)), "nnz": int(nnz), "ranks": "x".join(map(str, ranks)),
         "zipf": ",".join("%g" % z for z in (zipf or [0] * len(dims))), "prec": prec, "iters": int(iters)}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small exploratory decomposition (tens of thousands of entries, a few
        # invocations): latency and launches
        _case("hooi3-small", "hooi", (200, 150, 100), 20_000, (5, 5, 5), iters=3),
        # an ordinary three-mode decomposition at the usual rank 10
        _case("hooi3-mid", "hooi", (2003, 1501, 997), 2_000_000, (10, 10, 10), iters=2),
        # one long mode and skewed slices (users x items x contexts)
        _case("hooi3-large", "hooi", (300_000, 8_000, 4_001), 40_000_000, (10, 10, 10), (0.4, 0.4, 0.4), iters=2),
        # four modes, Khat = 1000, in the precision form (BF16 tiles and Gram
        # operands, then a refining FP32 invocation)
        _case("hooi4-bf16", "hooi", (50_000, 601, 150, 97), 10_000_000, (10, 10, 10, 10),
              (0.3, 0.3, 0.3, 0.3), prec="bf16", iters=2),
        # a small tensor's penultimate matrices, ragged sizes and ranks
        _case("ttm3-small", "ttm", (1201, 701, 89), 150_001, (7, 12, 5), (0.6, 0.8, 0.4)),
        # heavy-tailed interaction data: 1e8 draws, Zipf 1.1 in every mode
        _case("ttm3-zipf", "ttm", (1_000_000, 500_000, 200_000), 100_000_000, (10, 10, 10), (1.1, 1.1, 1.1)),
        # one flat mode (Zipf 0.8) of 4e6 rows: factor rows gathered from far memory
        _case("ttm3-flat", "ttm", (4_000_000, 4_000_000, 2_000_000), 200_000_000, (10, 10, 10), (0.8, 1.2, 1.5)),
        # four modes, Khat = 1000
        _case("ttm4-zipf", "ttm", (400_000, 200_000, 20_000, 5_000), 20_000_000, (10, 10, 10, 10),
              (0.9, 1.1, 1.3, 0.7)),
        # ranks above 16 (the shape no matrix-core kernel takes)
        _case("ttm3-wide", "ttm", (100_000, 50_000, 8_009), 8_000_000, (20, 24, 18), (0.8, 0.9, 0.6)),
        # completion of a small ratings-like tensor, odd ranks
        _case("fit3-small", "fit", (1_900, 801, 60), 200_003, (8, 7, 5), (0.7, 0.7, 0.3)),
        # completion with the embedding-sized factors of recommender data
        _case("fit3-large", "fit", (500_000, 500_000, 50_000), 50_000_000, (16, 16, 16), (1.0, 1.0, 1.0)),
        # a new tensor of 2e7 entries up to its first penultimate matrices
        _case("ingest3", "ingest", (200_000, 100_000, 40_000), 20_000_000, (10, 10, 10), (0.9, 0.9, 0.9)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["hooi", "hooi", "ttm", "ttm", "fit", "ingest"])
    N = rng.choice([3, 3, 3, 4])
    if path == "ttm" and rng.random() < 0.15:
        N = rng.choice([2, 5])
    if path == "hooi":
        # one long mode; the others short enough for the planted model to stand
        # out against single entries (nnz >= 15 sqrt(product of the dims))
        nnz = _log_int(rng, 2e4, 3e7) if N == 3 else _log_int(rng, 2e5, 8e6)
        dims = [max(60, min(int(nnz / rng.uniform(50, 400)), 300_000 if N == 3 else 50_000))]
        each = ((nnz / 15) ** 2 / dims[0]) ** (1 / (N - 1))
        dims += [max(24, min(int(each * rng.uniform(0.6, 1.0)), dims[0])) for _ in range(N - 1)]
        dims = [dims[n] for n in rng.sample(range(N), N)]
        z = [round(rng.uniform(0.0, 0.5), 2)] * N
        K = rng.choice([5, 8, 10, 10]) if N == 3 else rng.choice([4, 6, 10])
        ranks = [K] * N
        return _case("", path, dims, nnz, ranks, z, prec=rng.choice(["fp32", "fp32", "bf16"]), iters=rng.randint(1, 3))
    if path == "ttm":
        nnz = _log_int(rng, 1e5, 1e8 if N <= 3 else 1.5e7 if N == 4 else 1e6)
        dims = [_log_int(rng, 50, 2e6 if N <= 3 else 3e5) for _ in range(N)]
        if N == 3 and rng.random() < 0.2:
            ranks = [rng.randint(12, 24) for _ in range(N)]
            nnz = min(nnz, 8_000_000)
        else:
            ranks = [rng.choice([10, 10, rng.randint(2, 16)]) if N <= 3 else rng.randint(2, 10 if N == 4 else 5)
                     for _ in range(N)]
        z = [round(rng.uniform(0.5, 1.5), 2) for _ in range(N)]
        dims = [max(d, k) for d, k in zip(dims, ranks)]
        return _case("", path, dims, nnz, ranks, z, prec=rng.choice(["fp32", "fp32", "bf16"]) if N in (3, 4) else "fp32")
    if path == "fit":
        N = 3 if rng.random() < 0.85 else 4
        nnz = _log_int(rng, 1e5, 5e7) if N == 3 else _log_int(rng, 1e5, 1e6)
        dims = [_log_int(rng, 60, 5e5 if N == 3 else 1e4) for _ in range(N)]
        ranks = [rng.randint(2, 16 if N == 3 else 5) for _ in range(N)]
        return _case("", path, dims, nnz, ranks, [round(rng.uniform(0.0, 1.0), 2) for _ in range(N)])
    nnz = _log_int(rng, 1e5, 2e7 if N == 3 else 8e6)
    dims = [_log_int(rng, 100, 3e5 if N == 3 else 5e4) for _ in range(N)]
    ranks = [rng.randint(2, 10) for _ in range(N)]
    return _case("", "ingest", dims, nnz, ranks, [round(rng.uniform(0.3, 1.2), 2) for _ in range(N)])


# ---- inputs --------------------------------------------------------------------------------------

def _ints(s):
    return tuple(int(x) for x in s.split("x"))


def _zipf(case):
    return tuple(float(x) for x in case["zipf"].split(","))


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) % (1 << 40)) * 64 + stream)
    return g


def _coords(case, seed):
    """One int32 coordinate array per mode: Zipf ranks mapped through a random
    permutation.  The seed picks the permutation; the ranks are the case's own,
    so every seed has the same number of nonempty slices (rows of Y)."""
    nnz = case["nnz"]
    out = []
    for n, (L, s) in enumerate(zip(_ints(case["dims"]), _zipf(case))):
        perm = torch.randperm(L, generator=_gen(seed, n), device=DEV).to(torch.int32)
        g = _gen(0, 40 + n)
        # whole-number weights: their running sums do not depend on the order of the additions
        w = (torch.arange(1, L + 1, device=DEV, dtype=torch.float64) ** -s * 2.0 ** 38).long()
        cdf = torch.cumsum(w, 0).double()
        idx = torch.empty(nnz, dtype=torch.int32, device=DEV)
        for a in range(0, nnz, 1 << 25):
            b = min(a + (1 << 25), nnz)
            u = torch.rand(b - a, generator=g, device=DEV, dtype=torch.float64)
            idx[a:b] = perm[torch.searchsorted(cdf, u * cdf[-1]).clamp_(max=L - 1)]
        out.append(idx)
    return out


def _lognormal(nnz, seed):
    return torch.randn(nnz, generator=_gen(seed, 20), device=DEV).exp_()


def _factors(case, seed):
    """FP64 Gaussian factors with columns of about unit norm."""
    return [torch.randn(L, K, generator=_gen(seed, 30 + n), device=DEV, dtype=torch.float64) / math.sqrt(L)
            for n, (L, K) in enumerate(zip(_ints(case["dims"]), _ints(case["ranks"])))]


def _planted(case, idx, seed):
    """Values of a planted model (a sum of K rank-one terms of falling strength)
    plus noise, and orthonormal starting factors that overlap its factors."""
    dims, ranks = _ints(case["dims"]), _ints(case["ranks"])
    K = min(ranks)
    A = [3 ** 0.5 * (2 * torch.rand(L, K, generator=_gen(seed, 10 + n), device=DEV) - 1) for n, L in enumerate(dims)]
    w = 0.9 ** torch.arange(K, device=DEV, dtype=torch.float32)
    nnz = case["nnz"]
    vals = 0.1 * torch.randn(nnz, generator=_gen(seed, 20), device=DEV)
    for a in range(0, nnz, 1 << 23):
        b = min(a + (1 << 23), nnz)
        p = w.expand(b - a, K)
        for n in range(len(dims)):
            p = p * A[n][idx[n][a:b].long()]
        vals[a:b] += p.sum(1)
    F0 = []
    for n, (L, k) in enumerate(zip(dims, ranks)):
        S = torch.randn(L, k, generator=_gen(seed, 30 + n), device=DEV, dtype=torch.float64)
        S[:, :K] = 0.7 * S[:, :K] + A[n].double()
        F0.append(torch.linalg.qr(S)[0].contiguous())
    return vals, F0


def _context(case, idx, vals, **opt):
    ctx = tk.TuckerContext(0, prec=case["prec"], **opt)
    ctx.load_coo(idx, vals, _ints(case["dims"]))
    ctx.set_ranks(_ints(case["ranks"]))
    return ctx


def _fit_inputs(case, seed):
    dims, ranks = _ints(case["dims"]), _ints(case["ranks"])
    idx = _coords(case, seed)
    targets = torch.randn(case["nnz"], generator=_gen(seed, 20), device=DEV)
    core = torch.randn(math.prod(ranks), generator=_gen(seed, 21), device=DEV) / math.sqrt(math.prod(ranks) / 16)
    F = [0.5 * torch.randn(L, K, generator=_gen(seed, 30 + n), device=DEV)
         for n, (L, K) in enumerate(zip(dims, ranks))]
    return idx, targets, core, F


def prepare(case, seed):
    path = case["path"]
    s = {"case": case}
    if path == "fit":
        idx, s["targets"], core, F = _fit_inputs(case, seed)
        s["ctx"] = tk.TuckerContext(0)
        s["ctx"].load_obs(idx, _ints(case["dims"]), _ints(case["ranks"]))
        s["core"] = core.requires_grad_()
        s["F"] = [f.requires_grad_() for f in F]
        return s
    idx = _coords(case, seed)
    if path == "hooi":
        vals, s["F0"] = _planted(case, idx, seed)
        s["ctx"] = _context(case, idx, vals)
        s["F"] = [torch.empty_like(f) for f in s["F0"]]
        s["one"] = torch.ones((), dtype=torch.float64, device=DEV)
        return s
    vals = _lognormal(case["nnz"], seed)
    F = _factors(case, seed)
    if path == "ttm":
        s["ctx"] = _context(case, idx, vals)
        for n, f in enumerate(F):
            s["ctx"].set_factor(n, f)
        return s
    s.update(ctx=tk.TuckerContext(0), idx=idx, vals=vals, F=F)
    return s


# ---- one pass -------------------------------------------------------------------------------------

def run(s):
    case, ctx = s["case"], s["ctx"]
    path = case["path"]
    N = len(_ints(case["dims"]))
    if path == "hooi":
        for n, f in enumerate(s["F0"]):
            ctx.set_factor(n, f)
        fits = ctx.hooi_iterate(case["iters"])
        core, fit = ctx.core()
        # the factors go on as FP32 embeddings, the precision they are computed
        # to, their columns' signs (free in an SVD) those of the starting factors
        F, core = [], torch.from_numpy(core).to(DEV)
        for n in range(N):
            f = ctx.get_factor(n, out=s["F"][n])
            sign = torch.copysign(s["one"], (f * s["F0"][n]).sum(0))
            F.append((f * sign).float())
            core = core * sign.reshape([-1 if j == n else 1 for j in range(N)])
        if case["prec"] == "bf16":   # the precision form's results, kept in its type; earlier fits are not exact
            return {"fit": fits[-1], "core": core.bfloat16(), "factors": [f.bfloat16() for f in F]}
        return {"fits": fits, "fit": fit, "core": core.float(), "factors": F}
    if path == "ttm":
        return [dict(zip(("Y", "rows"), ctx.ttm_chain(n, device=True))) for n in range(N)]
    if path == "fit":
        model = tk.TuckerEval.apply(ctx, s["core"], *s["F"])
        loss = 0.5 * (model - s["targets"]).square().sum()
        grads = torch.autograd.grad(loss, [s["core"]] + s["F"])
        return {"model": model.detach(), "loss": loss.detach(), "grads": list(grads)}
    ctx.load_coo(s["idx"], s["vals"], _ints(case["dims"]))
    ctx.set_ranks(_ints(case["ranks"]))
    for n, f in enumerate(s["F"]):
        ctx.set_factor(n, f)
    out = [dict(zip(("Y", "rows"), ctx.ttm_chain(n, device=True))) for n in range(N)]
    m, norm_sq = ctx.tensor_info()
    return {"ttm": out, "m": m, "norm": math.sqrt(norm_sq)}


# ---- the work of one pass -------------------------------------------------------------------------

def _expected(case):
    """Expected distinct coordinates and nonempty slices per mode of the draws,
    from the marginals (ranks grouped in bins of nearly equal probability)."""
    dims, zipf, nnz = _ints(case["dims"]), _zipf(case), case["nnz"]
    bins = {2: 256, 3: 64, 4: 28, 5: 14}.get(len(dims), 10)
    R, cnt, prob = [], np.ones(1), np.ones(1)
    for L, s in zip(dims, zipf):
        p = np.arange(1, L + 1, dtype=np.float64) ** -s
        p /= p.sum()
        R.append(float(-np.expm1(-nnz * p).sum()))
        edges = np.unique(np.round(np.geomspace(1, L + 1, bins + 1)).astype(np.int64)) - 1
        c = np.diff(edges).astype(np.float64)
        q = np.add.reduceat(p, edges[:-1]) / c
        cnt, prob = (cnt[:, None] * c).ravel(), (prob[:, None] * q).ravel()
    return float((cnt * -np.expm1(-nnz * prob)).sum()), R


def work(case):
    dims, ranks, N = _ints(case["dims"]), _ints(case["ranks"]), len(_ints(case["dims"]))
    nnz = case["nnz"]
    m, R = _expected(case)
    khat = [math.prod(ranks) // k for k in ranks]
    if case["path"] == "fit":
        m = nnz   # observations are never merged
    ttm_b = ttm_f = 0.0
    for n in range(N):
        ttm_b += 4 * m * N + 4 * R[n] * khat[n] + 4 * sum(dims[j] * ranks[j] for j in range(N) if j != n)
        last = ranks[N - 1] if n < N - 1 else ranks[N - 2]
        ttm_f += m * (2 * khat[n] + khat[n] // last)
    fac = sum(L * K for L, K in zip(dims, ranks))
    if case["path"] == "ttm":
        return {"bytes": ttm_b, "flops": ttm_f}
    if case["path"] == "ingest":
        return {"bytes": 4 * nnz * (N + 1) + 4 * m * (N + 1) + 4 * N * N * m + ttm_b, "flops": ttm_f}
    if case["path"] == "hooi":
        svd_f = sum(R[n] * khat[n] * (khat[n] + 2 * ranks[n]) for n in range(N))
        one_b = ttm_b + 8 * fac
        return {"bytes": case["iters"] * one_b + 2 * 8 * fac, "flops": case["iters"] * (ttm_f + svd_f)}
    fwd_f = m * (2 * khat[N - 1] + 2 * ranks[0])
    grad_f = sum(2 * R[n] * khat[n] * ranks[n] for n in range(N))
    return {"bytes": 2 * 4 * m * (N + 1) + 3 * 4 * fac, "flops": fwd_f + ttm_f + grad_f}


# ---- the same in 64 bits --------------------------------------------------------------------------

def _add_rows(Y, at, p):
    """Y[at] += p, the runs of equal rows (at ascending) summed first, up to 512 at a time."""
    part = torch.arange(len(at), device=DEV) // 512
    key, counts = torch.unique_consecutive(at * len(at) + part, return_counts=True)
    Y.index_add_(0, key // len(at), torch.segment_reduce(p, "sum", lengths=counts, axis=0, unsafe=True))


def _ttm64(idx, vals, F, dims, n):
    """Y_(n) over the nonempty slices: first remaining mode fastest."""
    key, order = torch.sort(idx[n])
    rows, at = torch.unique_consecutive(key, return_inverse=True)
    others = [j for j in range(len(dims)) if j != n]
    khat = math.prod(F[j].shape[1] for j in others)
    Y = torch.zeros(len(rows), khat, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // khat)
    for a in range(0, len(vals), step):
        e = order[a:a + step]
        p = vals[e].double()[:, None]
        for j in others:
            p = (F[j][idx[j][e].long()][:, :, None] * p[:, None, :]).flatten(1)
        _add_rows(Y, at[a:a + step], p)
    return Y, rows


def _hooi64(case, seed):
    dims, ranks, N = _ints(case["dims"]), _ints(case["ranks"]), len(_ints(case["dims"]))
    idx = _coords(case, seed)
    vals, F0 = _planted(case, idx, seed)
    F = list(F0)
    # repeated coordinates are one entry of the tensor
    key = torch.zeros(len(vals), dtype=torch.long, device=DEV)
    for L, i in zip(dims, idx):
        key = key * L + i.long()
    key, inv = torch.unique(key, return_inverse=True)
    merged = torch.zeros(len(key), dtype=torch.float64, device=DEV).index_add_(0, inv, vals.double())
    norm = merged.norm()
    idx = []
    for L in reversed(dims):
        idx.insert(0, (key % L).int())
        key = key // L
    fits = []
    for _ in range(case["iters"]):
        for n in range(N):
            Y, rows = _ttm64(idx, merged, F, dims, n)
            lam, V = torch.linalg.eigh(Y.T @ Y)
            V = V[:, -ranks[n]:].flip(1)
            U = torch.linalg.qr(Y @ V)[0]
            F[n] = torch.zeros(dims[n], ranks[n], dtype=torch.float64, device=DEV)
            F[n][rows.long()] = U
        G = F[N - 1][rows.long()].T @ Y
        fits.append(float(1 - torch.sqrt((norm ** 2 - G.norm() ** 2).clamp(min=0)) / norm))
    core = G.reshape([ranks[N - 1]] + [ranks[j] for j in reversed(range(N - 1))]).permute(*reversed(range(1, N)), 0)
    for n in range(N):
        sign = torch.sign((F[n] * F0[n]).sum(0))
        F[n] = F[n] * sign
        core = core * sign.reshape([-1 if j == n else 1 for j in range(N)])
    if case["prec"] == "bf16":
        return {"fit": fits[-1], "core": core, "factors": F}
    return {"fits": fits, "fit": fits[-1], "core": core, "factors": F}


def exact(case, seed):
    dims, ranks, N = _ints(case["dims"]), _ints(case["ranks"]), len(_ints(case["dims"]))
    nnz, cells = case["nnz"], math.prod(ranks)
    if case["path"] == "hooi":
        if nnz * cells > 1.2e11 or math.prod(dims) >= 1 << 62:
            return None
        return _hooi64(case, seed)
    if case["path"] == "fit":
        if nnz * cells > 4e11:
            return None
        idx, targets, core, F = _fit_inputs(case, seed)
        return _fit64(idx, targets.double(), core.double(), [f.double() for f in F], ranks)
    if nnz * sum(cells // k for k in ranks) > 1e11:
        return None
    idx = _coords(case, seed)
    vals = _lognormal(nnz, seed)
    F = _factors(case, seed)
    out = [dict(zip(("Y", "rows"), _ttm64(idx, vals, F, dims, n))) for n in range(N)]
    if case["path"] == "ttm":
        return out
    return {"ttm": out, "m": None, "norm": None}


def _fit64(idx, targets, core, F, ranks):
    N = len(ranks)
    G = core.reshape(tuple(reversed(ranks)))       # last index of the core slowest
    G = G.permute(*reversed(range(N))).contiguous()
    model = torch.empty_like(targets)
    dG = torch.zeros(math.prod(ranks), dtype=torch.float64, device=DEV)
    dF = [torch.zeros_like(f) for f in F]
    step = max(1, (1 << 27) * ranks[0] // math.prod(ranks))
    for a in range(0, len(targets), step):
        rows = [F[j][idx[j][a:a + step].long()] for j in range(N)]
        with torch.enable_grad():
            g = G.reshape(-1).clone().requires_grad_()
            r = [x.clone().requires_grad_() for x in rows]
            t = r[0] @ g.reshape(ranks[0], -1)     # obs x (the other modes, in order)
            for j in range(1, N):
                t = (t.reshape(len(t), ranks[j], -1) * r[j][:, :, None]).sum(1)
            y = t.reshape(-1)
            d = torch.autograd.grad(0.5 * (y - targets[a:a + step]).square().sum(), [g] + r)
        model[a:a + step] = y.detach()
        dG += d[0]
        for j in range(N):
            key, order = torch.sort(idx[j][a:a + step].long())
            _add_rows(dF[j], key, d[1 + j][order])
    dcore = dG.reshape(tuple(ranks)).permute(*reversed(range(N))).reshape(-1)
    return {"model": model, "loss": 0.5 * (model - targets).square().sum(), "grads": [dcore] + dF}
