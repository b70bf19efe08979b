"""What a user of this library has it do, as measurable cases over the public entry points.

Decode-time projection (one call per decode step, from one row to thousands, greedy and top-k, uniform and
skewed batches, long synthetic candidate lists and short learned ones), the full-vocabulary projection (few
rows, ragged sizes, and the long recording pass in front of the training of the clusters), the batch-union
form, a beam-search step, and the training of the clusters.  Sizes are those of workloads.CONFIGS, of the
benchmark's decode loop, cluster sweep and cluster training, and of 20 sentences x beam 2; everything is
seeded and made on the GPU.
"""
import math

import numpy as np
import torch

import paper_2208_06874_amd as P

MAX_SLAB_BYTES = 34e9     # packed lists of the largest listed index (31 GB) and some padding
MAX_FLOPS = 8.5e12        # the recording pass
NOISE = 0.3               # of a row around its centroid, as in workloads.CONFIGS


def listed():
    sweep = dict(d=1024, V=250000, K=1000, lo=10000, hi=20000, rows="uniform", sizes="uniform")
    return [
        # greedy decoding of one sentence: the smallest call, all latency and launches
        dict(sweep, name="greedy_1", kind="project", N=1, k=1),
        # one sentence with five beams
        dict(sweep, name="beam_5", kind="project", N=5, k=5),
        # a small model: 16 rows against 32 clusters of about 2,000 tokens
        dict(name="small_16", kind="project", d=512, V=32000, K=32, N=16, k=4, lo=1800, hi=2200, rows="uniform", sizes="uniform"),
        # 8 sentences x beam 8
        dict(name="mid_64", kind="project", d=1024, V=128000, K=200, N=64, k=8, lo=5000, hi=8000, rows="uniform", sizes="uniform"),
        # the benchmark's headline: a serving batch of 32 sentences x beam 8 on a multilingual vocabulary
        dict(sweep, name="large_256", kind="project", N=256, k=8),
        # greedy decoding of a large batch
        dict(sweep, name="greedy_1024", kind="project", N=1024, k=1),
        # 512 sentences x beam 8 whose rows crowd into a few clusters, lists from short to long
        dict(name="skewed_4096", kind="project", d=1536, V=250000, K=500, N=4096, k=8, lo=2000, hi=40000, rows="zipf", sizes="loguniform"),
        # a beam-search step on learned clusters: short lists, the projection and the search step after it
        dict(name="learned_beam_64", kind="beam", d=1024, V=250000, K=1000, N=64, B=8, k=8, lo=100, hi=900),
        # 20 sentences x beam 2, the batch-union form on learned clusters (union: a few percent to a sixth of V)
        dict(name="union_40", kind="union", d=1024, V=250000, K=1300, N=40, k=2, lo=300, hi=1500),
        # the plain projection at sizes that fill no tile: 333 rows, a vocabulary and a width off every power of two
        dict(name="full_ragged_333", kind="full", d=1000, V=150001, N=333, k=5),
        # recording pass in front of the training: the top 3 tokens of every recorded vector
        dict(name="record_16384", kind="full", d=1024, V=250000, N=16384, k=3),
        # training of the clusters on recorded vectors, 20 iterations
        dict(name="kmeans_131072", kind="kmeans", d=1024, n=131072, K=1000, iters=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    return rng.choice((512, 768, 1024, 1024, 1536, 8 * rng.randint(32, 192)))


def draw(rng):
    kind = rng.choice(("project", "project", "project", "full", "full", "beam", "union", "kmeans"))
    d = _width(rng)
    V = _log_int(rng, 32000, 250000)
    if kind == "kmeans":
        K = _log_int(rng, 32, 1300)
        n = _log_int(rng, 3000, 131072)
        return dict(kind=kind, d=d, n=n, K=K, iters=rng.randint(3, 20))
    if kind == "full":
        N = _log_int(rng, 1, 16384)
        N = max(1, min(N, int(MAX_FLOPS / (2.0 * d * V))))
        return dict(kind=kind, d=d, V=V, N=N, k=rng.randint(1, 8))
    K = _log_int(rng, 32, 1300)
    if kind in ("beam", "union"):
        hi = max(200, _log_int(rng, V // 500, V // 100))
        N = _log_int(rng, 2, 256)
        if kind == "union":
            return dict(kind=kind, d=d, V=V, K=K, N=N, k=rng.randint(1, 8), lo=max(50, hi // 6), hi=hi)
        B = rng.choice((1, 2, 4, 5, 8))
        return dict(kind=kind, d=d, V=V, K=K, N=max(1, N // B) * B, B=B, k=max(B, rng.randint(1, 8)), lo=max(50, hi // 6), hi=hi)
    hi = _log_int(rng, V // 40, V // 8)
    sizes = rng.choice(("uniform", "loguniform"))
    lo = hi // 2 if sizes == "uniform" else hi // 16
    mean = (lo + hi) / 2 if sizes == "uniform" else (hi - lo) / math.log(hi / lo)
    K = max(16, min(K, int(MAX_SLAB_BYTES / (mean * 2 * _padded(d)))))
    N = _log_int(rng, 1, 4096)
    return dict(kind=kind, d=d, V=V, K=K, N=N, k=rng.randint(1, 8), lo=lo, hi=hi, rows="zipf" if N >= 64 and rng.random() < 0.4 else "uniform", sizes=sizes)


# ---------------------------------------------------------------- inputs
def _padded(d):
    return (d + 255) // 256 * 256


def _zipf(K):
    p = np.arange(1, K + 1, dtype=np.float64) ** -1.1
    return p / p.sum()


def _rows(g, C, N, weights=None):
    """N hidden rows: a centroid each, plus noise."""
    K, d = C.shape
    if weights is None:
        q = torch.randint(0, K, (N,), generator=g, device="cuda")
    else:
        w = torch.from_numpy(weights).float().cuda()[torch.randperm(K, generator=g, device="cuda")]
        q = torch.multinomial(w, N, replacement=True, generator=g)
    return (C[q].float() + NOISE * torch.randn((N, d), generator=g, device="cuda")).half()


def _model(g, d, V):
    W = torch.randn((d, V), generator=g, device="cuda", dtype=torch.float16).mul_(d ** -0.5)
    b = torch.randn((V,), generator=g, device="cuda").mul_(math.sqrt(0.1)).half()
    return W, b


def _lists(g, case, W, b, C):
    """Active sets of about the configured sizes as the ascending lists vp_build takes: the tokens that the
    centroid itself scores highest, filled up with random tokens (lists of learned clusters: scored ones only)."""
    (K, d), V = C.shape, W.shape[1]
    u = torch.rand((K, 1), generator=g, device="cuda")
    lo, hi = case["lo"], case["hi"]
    size = lo * (hi / lo) ** u if case.get("sizes") == "loguniform" else lo + (hi - lo) * u
    scored = size * (1.0 if case["kind"] in ("beam", "union") else 0.1)
    spread = torch.sqrt(C.float().square().sum(1, keepdim=True) / d + 0.1)
    bar = spread * math.sqrt(2.0) * torch.erfinv(1.0 - 2.0 * scored / V)
    member = (C @ W + b).float() > bar
    member |= torch.rand((K, V), generator=g, device="cuda") < (size - scored) / V
    member[:, 0] = True       # (no empty list)
    off = np.zeros(K + 1, np.int64)
    off[1:] = member.sum(1).cumsum(0).cpu().numpy()
    return off, member.nonzero()[:, 1].to(torch.int32).cpu().numpy()


def _training(case, seed):
    g = torch.Generator("cuda")
    g.manual_seed(seed)
    n, d, K = case["n"], case["d"], case["K"]
    X = _rows(g, torch.randn((K, d), generator=g, device="cuda").half(), n)
    return X, X[torch.randperm(n, generator=g, device="cuda")[:K]].clone()


def _inputs(case, seed):
    """Weights, bias, centroids, active sets, hidden rows and (beam search) scores of the hypotheses."""
    g = torch.Generator("cuda")
    g.manual_seed(seed)
    kind, d, N = case["kind"], case["d"], case["N"]
    W, b = _model(g, d, case["V"])
    C = torch.randn((case.get("K", 1), d), generator=g, device="cuda").half()
    if kind == "full":       # an index for the plain projection alone: one cluster with one token
        off, ids = np.array([0, 1], np.int64), np.array([0], np.int32)
    else:
        off, ids = _lists(g, case, W, b, C)
    centers = torch.randn((1000, d), generator=g, device="cuda").half() if kind == "full" else C
    hidden = _rows(g, centers, N, _zipf(C.shape[0]) if case.get("rows") == "zipf" else None)
    scores = torch.randn((N,), generator=g, device="cuda") - 20.0 if kind == "beam" else None
    return W, b, C, off, ids, hidden, scores


def prepare(case, seed):
    kind, d = case["kind"], case["d"]
    if kind == "kmeans":
        X, start = _training(case, seed)
        ws = torch.empty(P.vp.vp_kmeans_workspace_bytes(case["n"], d, case["K"]), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, X=X, start=start, iters=case["iters"], ws=ws)
    N, k = case["N"], case["k"]
    W, b, C, off, ids, hidden, scores = _inputs(case, seed)
    index = P.vp_build(W, b, C, off, ids, k_max=max(8, k))
    st = dict(kind=kind, index=index, hidden=hidden, k=k)
    # what a decode loop keeps from step to step: its outputs and its workspace
    st["ids"] = torch.empty((N, k), dtype=torch.int32, device="cuda")
    st["logp"] = torch.empty((N, k), dtype=torch.float32, device="cuda")
    st["cluster"] = torch.empty((N,), dtype=torch.int32, device="cuda")
    need = P.vp.vp_union_workspace_bytes(index, N) if kind == "union" else P.vp.vp_workspace_bytes(index, N)
    st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    if kind == "union":
        st["size"] = torch.zeros((1,), dtype=torch.int32, device="cuda")
    if kind == "beam":
        st["B"] = case["B"]
        st["scores"] = scores
        st["out"] = (torch.empty_like(scores), torch.empty((N,), dtype=torch.int32, device="cuda"),
                     torch.empty((N,), dtype=torch.int32, device="cuda"))
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    kind = st["kind"]
    if kind == "kmeans":
        centroids = st["start"].clone()
        assign, _counts = P.vp.vp_kmeans(st["X"], centroids, st["iters"], workspace=st["ws"])
        return centroids, assign      # (the counts are assign's histogram)
    if kind == "full":
        return P.vp_project_full(st["index"], st["hidden"], st["k"], out_ids=st["ids"], out_logp=st["logp"], workspace=st["ws"])
    if kind == "union":
        return P.vp.vp_project_union(st["index"], st["hidden"], st["k"], out_ids=st["ids"], out_logp=st["logp"],
                                     out_cluster=st["cluster"], out_union_size=st["size"], workspace=st["ws"])
    ids, logp, cluster = P.vp_project(st["index"], st["hidden"], st["k"], out_ids=st["ids"], out_logp=st["logp"],
                                      out_cluster=st["cluster"], workspace=st["ws"])
    if kind == "beam":
        return (ids, logp, cluster) + tuple(P.vp.vp_beam_step(ids, logp, st["scores"], st["B"], out=st["out"]))
    return ids, logp, cluster


# ---------------------------------------------------------------- what a pass cannot do without
def _mean_list(case):
    lo, hi = case["lo"], case["hi"]
    return (hi - lo) / math.log(hi / lo) if case.get("sizes") == "loguniform" else (lo + hi) / 2


def work(case):
    d = case["d"]
    if case["kind"] == "kmeans":
        n, K = case["n"], case["K"]
        return dict(bytes=n * d * 2.0 + K * d * 4.0 + n * 4.0 + K * 4.0,
                    flops=2.0 * n * K * d * (case["iters"] + 1) + n * d * case["iters"])
    V, N, k = case["V"], case["N"], case["k"]
    io = N * (2.0 * d + 8.0 * k)
    if case["kind"] == "full":
        return dict(bytes=V * (2.0 * d + 2.0) + io, flops=2.0 * N * V * d)
    # the columns of every token that some row's cluster lists, once; every row against its own list
    K, n = case["K"], _mean_list(case)
    p = _zipf(K) if case.get("rows") == "zipf" else np.full(K, 1.0 / K)
    occupied = float((1.0 - (1.0 - p) ** N).sum())
    union = V * (1.0 - (1.0 - n / V) ** occupied)
    row_tokens = union if case["kind"] == "union" else n
    return dict(bytes=union * (2.0 * d + 2.0) + K * 2.0 * d + io + N * 4.0, flops=2.0 * N * d * (K + row_tokens))


def tolerance(case):
    if case["kind"] == "kmeans":
        # against the same iterations with scores in fp64: centroids up to 2.3e-4 (norm) and 0.021 (largest), where a
        # few vectors halfway between two centroids went to the other one; 1e-5 of the memberships, more with few clusters
        return dict(rel=1e-3, max=0.1, differ=1e-3)
    # log-probs against fp64 logits: up to 1.9e-7 (norm) and 6.3e-7 (largest); ids and clusters equal but for ties in fp32
    return dict(rel=2e-6, max=4e-6, differ=1e-3)


# ---------------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    """The log-probabilities (and a beam step's scores) in 64 bits.  Whole numbers have no rounding; the training has
    no value of its own to compare with, since a vector halfway between two centroids goes to either."""
    if case["kind"] == "kmeans":
        return None
    W, b, C, off, ids, hidden, scores = _inputs(case, seed)
    kind, V, k = case["kind"], case["V"], case["k"]
    W, b, h = W.double(), b.double(), hidden.double()
    member = None
    if kind != "full":
        C = C.double()
        cluster = (C.square().sum(1) - 2.0 * (h @ C.T)).argmin(1)
        counts = torch.from_numpy(np.diff(off)).cuda()
        owner = torch.repeat_interleave(torch.arange(len(off) - 1, device="cuda"), counts)
        member = torch.zeros((len(off) - 1, V), dtype=torch.bool, device="cuda")
        member[owner, torch.from_numpy(ids).cuda().long()] = True
        if kind == "union":
            member[:] = member[cluster.unique()].any(0)
    logp = []
    for r in range(0, h.shape[0], 512):
        z = h[r:r + 512] @ W + b
        if member is not None:
            z.masked_fill_(~member[cluster[r:r + 512]], -math.inf)
        logp.append(z.topk(k, 1).values - z.logsumexp(1, keepdim=True))
    logp = torch.cat(logp)
    if kind == "full":
        return None, logp
    if kind == "union":
        return None, logp, None, None
    if kind == "beam":
        sums = (scores.double()[:, None] + logp).reshape(-1, case["B"] * k)
        return None, logp, None, sums.topk(case["B"], 1).values.reshape(-1), None, None
    return None, logp, None
