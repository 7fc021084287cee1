"""Performance cases: searches, index construction and model training of the
library at the sizes users run, through its public Python entry points.

A case is a dict of plain values. `prepare` builds what a program holds before
the call (an index over synthetic vectors, queries, output buffers), `run` is
one pass, `work` the bytes and operations that pass cannot do without, `exact`
the results in 64 bits by plain torch.

Vectors (seeded, drawn on the GPU): "sift" - non-negative integers 0..255 from
a mixture with heavy-tailed per-dimension spread; "gist" - values in [0, 1]
with Zipf-sized components and a decaying spread; "embed" - a power-law
spectrum, unit length (uneven lengths for the inner product).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2405_12497_amd import rabitq as rq

METRICS = {"l2": rq.RBQ_METRIC_L2, "ip": rq.RBQ_METRIC_IP, "cosine": rq.RBQ_METRIC_COSINE}
SCANS = {"auto": rq.RBQ_SCAN_AUTO, "mfma": rq.RBQ_SCAN_MFMA, "fp4": rq.RBQ_SCAN_MFMA_FP4}


def _search(name, data, n, dim, nlist, nq, nprobe, k, metric="l2", rot="fp32", scan="auto", bq=4,
            learned=False, host=False, graph=False):
    return {"name": name, "kind": "search", "data": data, "n": n, "dim": dim, "nlist": nlist, "nq": nq,
            "nprobe": nprobe, "k": k, "metric": metric, "rot": rot, "scan": scan, "bq": bq,
            "learned": learned, "host": host, "graph": graph}


def listed():
    return [
        # an interactive lookup: one query against a small index, latency only
        _search("one_query", "sift", 100_000, 128, 512, 1, 16, 10),
        # a service request with a few host-side queries, maximum inner product, odd sizes
        _search("ip_host_37", "embed", 200_003, 100, 1024, 37, 33, 10, metric="ip", host=True),
        # word-embedding lookups by cosine, a thousand at a time
        _search("cosine_1000", "embed", 400_000, 300, 2048, 1000, 48, 20, metric="cosine"),
        # 8-bit queries (the finest quantisation on offer) on a mid-sized batch
        _search("bq8_500", "sift", 300_000, 200, 1024, 500, 40, 10, bq=8),
        # throughput search of image descriptors, FP32 rotation and popcount scan
        _search("sift_10k", "sift", 1_000_000, 128, 4096, 10_000, 20, 10),
        # top-100 of wide image features in batches of 256, batched scan
        _search("gist_256", "gist", 1_000_000, 960, 4096, 256, 8, 100, rot="bf16x3", scan="mfma"),
        # an uneven mid-sized batch on text embeddings with the default kernel choice
        _search("embed_333", "embed", 1_000_000, 768, 4096, 333, 192, 10, rot="bf16x3"),
        # one query against every list: the scan's memory-bound end
        _search("embed_all_lists", "embed", 4_000_000, 768, 8192, 1, 8192, 10, rot="bf16x3"),
        # throughput search of text embeddings, fixed nprobe, batched scan
        _search("embed_10k", "embed", 2_000_000, 768, 4096, 10_000, 128, 10, rot="bf16x3", scan="mfma"),
        # the same over twice the vectors, with a per-query nprobe from the loaded model
        _search("embed_learned", "embed", 4_000_000, 768, 8192, 10_000, 384, 10, rot="bf16x3", scan="mfma",
                learned=True),
        # a new index: k-means, build, first answers
        {"name": "index_new", "kind": "index", "data": "sift", "n": 300_000, "dim": 128, "nlist": 1024,
         "iters": 5, "nq": 100, "nprobe": 16, "k": 10},
        # training the nprobe model on recorded features and labels
        {"name": "train", "kind": "train", "n": 65_536, "batch": 4096, "epochs": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.random()
    if what < 0.1:
        return {"kind": "train", "n": _log(rng, 5_000, 100_000), "batch": rng.choice([1024, 4096, 5000]),
                "epochs": rng.randint(1, 2)}
    n = _log(rng, 30_000, 1_000_000)
    nlist = max(64, min(4096, int(rng.uniform(1.5, 5) * math.sqrt(n))))
    if what < 0.2:
        dim = rng.choice([64, 96, 100, 128, 200, 256])
        return {"kind": "index", "data": rng.choice(["sift", "embed"]), "n": min(n, 300_000), "dim": dim,
                "nlist": min(nlist, 1024), "iters": rng.randint(1, 5), "nq": _log(rng, 1, 200),
                "nprobe": _log(rng, 1, 32), "k": _log(rng, 1, 50)}
    dim = rng.choice([48, 64, 96, 100, 128, 200, 256, 300, 384, 512, 768, 960, rng.randint(32, 1024)])
    bq = rng.choice([4, 4, 4, 4, 6, 8])
    scan = rng.choice(["auto", "mfma", "mfma", "fp4"])
    if bq > 4 and scan == "fp4":
        scan = "mfma"
    nq = _log(rng, 1, 10_000)
    nprobe = _log(rng, 1, min(nlist, 256))
    learned = rng.random() < 0.15
    if not learned and nq <= 16 and rng.random() < 0.3:
        nprobe = nlist
    c = _search("", rng.choice(["sift", "gist", "embed"]), n, dim, nlist, nq, nprobe, _log(rng, 1, 128),
                metric=rng.choice(["l2", "l2", "l2", "ip", "cosine"]), rot=rng.choice(["fp32", "bf16x3"]),
                scan=scan, bq=bq, learned=learned, host=rng.random() < 0.15, graph=rng.random() < 0.1)
    del c["name"]
    # no costlier than the largest listed case
    while c["nprobe"] > 1 and c["nq"] * c["nprobe"] * c["n"] // c["nlist"] * c["dim"] > 1.5e11:
        c["nprobe"] = c["nprobe"] // 2
    return c


# ---------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 16 + stream)
    return g


def _maker(case, seed):
    """draw(m, generator) -> m vectors of the case's distribution."""
    dim, g = case["dim"], _gen(seed, 0)
    dev = {"generator": g, "device": "cuda"}
    if case["data"] == "sift":
        scale = torch.exp(torch.randn(dim, **dev)) * 20.0
        means = (torch.randn(64, dim, **dev) * (2.0 * scale)).abs_() + 10.0

        def make(m, h):
            comp = torch.randint(0, 64, (m,), generator=h, device="cuda")
            x = torch.randn(m, dim, generator=h, device="cuda").mul_(scale).add_(means[comp])
            return x.round_().clamp_(0.0, 255.0)
    elif case["data"] == "gist":
        sigma = 0.25 * torch.arange(1, dim + 1, device="cuda", dtype=torch.float32) ** -0.5
        means = torch.rand(4096, dim, **dev) * 0.5 + 0.1
        cum = torch.cumsum(torch.arange(1, 4097, device="cuda", dtype=torch.float64) ** -1.1, 0)

        def make(m, h):
            u = torch.rand(m, generator=h, device="cuda", dtype=torch.float64) * cum[-1]
            comp = torch.searchsorted(cum, u).clamp_(max=4095)
            x = torch.randn(m, dim, generator=h, device="cuda").mul_(sigma).add_(means[comp])
            return x.clamp_(0.0, 1.0)
    else:
        lam = torch.arange(1, dim + 1, device="cuda", dtype=torch.float32) ** -0.5
        ip = case.get("metric") == "ip"

        def make(m, h):
            x = torch.randn(m, dim, generator=h, device="cuda").mul_(lam)
            x /= x.norm(dim=1, keepdim=True)
            if ip:
                x *= torch.exp(0.2 * torch.randn(m, 1, generator=h, device="cuda"))
            return x
    return make


def _vectors(case, seed):
    make, h = _maker(case, seed), _gen(seed, 1)
    n, blk = case["n"], 1 << 18
    data = torch.empty(n, case["dim"], device="cuda")
    for s in range(0, n, blk):
        data[s:s + blk] = make(min(blk, n - s), h)
    return data, make(case["nq"], _gen(seed, 2)).contiguous()


def _nearest(x, c):
    cn = (c * c).sum(1)
    out = torch.empty(x.shape[0], dtype=torch.int32, device="cuda")
    for s in range(0, x.shape[0], 1 << 17):
        out[s:s + (1 << 17)] = torch.addmm(cn, x[s:s + (1 << 17)], c.T, alpha=-2.0).argmin(1)
    return out


def _lists(data, nlist, unit):
    """IVF lists: two Lloyd rounds on a sample (integer sums, so that every make
    of one seed gives the same bits), then every row to its nearest centroid."""
    def rows(x):
        return x / x.norm(dim=1, keepdim=True).clamp_min(1e-20) if unit else x
    n = data.shape[0]
    take = torch.arange(min(n, 32 * nlist), device="cuda") * n // min(n, 32 * nlist)
    x = rows(data[take])
    c = x[torch.arange(nlist, device="cuda") * x.shape[0] // nlist].clone()
    scale = 2.0 ** 30 / max(1.0, float(x.abs().max()))
    for _ in range(2):
        a = _nearest(x, c).long()
        cnt = torch.zeros(nlist, dtype=torch.int64, device="cuda").index_add_(0, a, torch.ones_like(a))
        sums = torch.zeros(nlist, x.shape[1], dtype=torch.int64, device="cuda")
        sums.index_add_(0, a, (x.double() * scale).round_().long())
        c = torch.where(cnt[:, None] > 0, (sums.double() / scale / cnt.clamp_min(1)[:, None]).float(), c)
    assign = torch.cat([_nearest(rows(data[s:s + (1 << 17)]), c) for s in range(0, n, 1 << 17)])
    return c.contiguous(), assign


def _inputs(case, seed):
    data, queries = _vectors(case, seed)
    cent, assign = _lists(data, case["nlist"], case["metric"] == "cosine")
    return data, queries, cent, assign


def _model(seed):
    """Weights of an nprobe model: a spread of buckets around the upper half."""
    r = np.random.default_rng(seed)
    w1 = r.standard_normal((rq.MLP_IN, rq.MLP_HIDDEN)) * (0.5 / math.sqrt(rq.MLP_IN))
    w2 = r.standard_normal((rq.MLP_HIDDEN, rq.MLP_OUT)) * (1.0 / math.sqrt(rq.MLP_HIDDEN))
    b2 = -0.02 * (np.arange(rq.MLP_OUT) - 22.0) ** 2
    return np.concatenate([w1.ravel(), np.zeros(rq.MLP_HIDDEN), w2.ravel(), b2]).astype(np.float32)


def _train_inputs(case, seed):
    h = _gen(seed, 3)
    x = torch.randn(case["n"], rq.MLP_IN, generator=h, device="cuda")
    x[:, 1:64] = x[:, 1:64].abs().mul_(0.05).cumsum(1)   # growing log distance ratios
    t = torch.randn(rq.MLP_IN, generator=h, device="cuda") * 0.2
    s = x @ t
    s = (s - s.mean()) / s.std() * 6.0 + 16.0 + torch.randn(case["n"], generator=h, device="cuda")
    return x.contiguous(), s.round().clamp_(0, rq.MLP_OUT - 1).int()


class _State:
    pass


def prepare(case, seed):
    st = _State()
    st.case, st.seed = case, seed
    if case["kind"] == "train":
        st.feats, st.labels = _train_inputs(case, seed)
        st.index = rq.Index(8, 1)   # the handle that holds the model
        return st
    if case["kind"] == "index":
        st.data, st.queries = _vectors(case, seed)
        return st
    data, queries, cent, assign = _inputs(case, seed)
    st.index = rq.Index(case["dim"], case["nlist"], bq=case["bq"], metric=METRICS[case["metric"]], seed=seed,
                        rot_precision=rq.RBQ_ROT_BF16X3 if case["rot"] == "bf16x3" else rq.RBQ_ROT_FP32)
    dp = st.index.code_bits
    p, _ = np.linalg.qr(np.random.default_rng(seed).standard_normal((dp, dp)))
    st.index.build_rotation(data, cent, assign, np.ascontiguousarray(p))
    del data, assign
    if case["learned"]:
        rq.rbq_nprobe_model_set(st.index.h, _model(seed), 0.8)
    st.opts = {"scan_kernel": SCANS[case["scan"]], "use_learned_nprobe": case["learned"], "use_graph": case["graph"]}
    if case["host"]:
        st.queries = queries.cpu().numpy()
    else:
        st.queries = queries
        st.opts["out_ids"] = torch.empty(case["nq"], case["k"], dtype=torch.int64, device="cuda")
        st.opts["out_dists"] = torch.empty(case["nq"], case["k"], device="cuda")
    return st


def run(st):
    case = st.case
    if case["kind"] == "train":
        losses = rq.rbq_nprobe_model_train(st.index.h, st.feats, st.labels, epochs=case["epochs"],
                                           batch=case["batch"], seed=st.seed)
        return {"losses": losses, "weights": rq.rbq_nprobe_model_get(st.index.h)[0]}
    if case["kind"] == "index":
        cent, assign = rq.rbq_kmeans(st.data, case["nlist"], iters=case["iters"],
                                     sample=min(case["n"], 64 * case["nlist"]), seed=st.seed)
        index = rq.Index(case["dim"], case["nlist"], seed=st.seed)
        index.build(st.data, cent, assign)
        ids, dists, _ = index.search(st.queries, case["k"], min(case["nprobe"], case["nlist"]))
        index.close()
        return {"centroids": cent, "assign": assign, "ids": ids, "dists": dists}
    ids, dists, _ = st.index.search(st.queries, case["k"], case["nprobe"], **st.opts)
    return {"ids": ids, "dists": dists}


def work(case):
    if case["kind"] == "train":
        params, rows = rq.MLP_NPARAM, case["n"] * case["epochs"]
        steps = -(-case["n"] // case["batch"]) * case["epochs"]
        return {"bytes": rows * (rq.MLP_IN * 4 + 4) + steps * params * 4 * 7, "flops": rows * 6 * params}
    n, dim, nlist, nq, nprobe = (case[k] for k in ("n", "dim", "nlist", "nq", "nprobe"))
    dp = -(-dim // 64) * 64
    nprobe = min(nprobe, nlist) * (0.5 if case.get("learned") else 1)   # the model's mean is about half its cap
    probed = nlist * -math.expm1(nq * math.log1p(-nprobe / nlist)) if nprobe < nlist else nlist
    codes = probed * n / nlist
    # queries, centroids (raw and rotated), codes and factors, the results' raw vectors, outputs
    b = nq * dim * 4 + nlist * (dim + dp) * 4 + codes * (dp / 8 + 8) + nq * case["k"] * (dim * 4 + 12)
    f = 2 * nq * dim * nlist + 2 * nq * dim * dp + 2 * nq * nprobe * (n / nlist) * dp + 3 * nq * case["k"] * dim
    if case["kind"] == "index":
        rows = min(n, 64 * nlist)
        b += (case["iters"] * rows + 2 * n) * dim * 4 + n * (dim * 4 + dp / 8 + 20)
        f += 2 * dim * nlist * (case["iters"] * rows + n) + 2 * n * dim * dp
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """The k best of each query's probed lists in 64 bits (None for the ids,
    whose order at equal keys is the library's own, and where the model or a
    whole k-means run chooses the lists)."""
    if case["kind"] != "search" or case["learned"]:
        return None
    data, queries, cent, assign = _inputs(case, seed)
    nq, nprobe, k, nlist = case["nq"], case["nprobe"], case["k"], case["nlist"]
    dot = case["metric"] != "l2"

    def unit(x):
        return x / x.norm(dim=1, keepdim=True) if case["metric"] == "cosine" else x
    q, c = unit(queries.double()), cent.double()
    probe = torch.empty(nq, nprobe, dtype=torch.int64, device="cuda")
    for s in range(0, nq, 2048):
        d = -(q[s:s + 2048] @ c.T) if dot else (c * c).sum(1) - 2.0 * (q[s:s + 2048] @ c.T)
        probe[s:s + 2048] = torch.sort(d, dim=1, stable=True).indices[:, :nprobe]
    order = torch.sort(assign.long(), stable=True).indices
    off = [0] + torch.cumsum(torch.bincount(assign.long(), minlength=nlist), 0).tolist()
    by_list = torch.sort(probe.reshape(-1), stable=True)
    pairs, rank = by_list.indices // nprobe, by_list.indices % nprobe
    poff = [0] + torch.cumsum(torch.bincount(by_list.values, minlength=nlist), 0).tolist()
    best = torch.full((nq, nprobe, k), math.inf, dtype=torch.float64, device="cuda")
    for l in range(nlist):
        lo, hi = poff[l], poff[l + 1]
        if lo == hi or off[l] == off[l + 1]:
            continue
        x = unit(data[order[off[l]:off[l + 1]]].double())
        y = q[pairs[lo:hi]]
        d = -(y @ x.T) if dot else ((y * y).sum(1, keepdim=True) + (x * x).sum(1) - 2.0 * (y @ x.T)).clamp_min(0.0)
        m = min(k, d.shape[1])
        best[pairs[lo:hi], rank[lo:hi], :m] = torch.topk(d, m, dim=1, largest=False).values
    d = torch.topk(best.reshape(nq, -1), k, dim=1, largest=False).values
    return {"ids": None, "dists": -d if dot else d}
