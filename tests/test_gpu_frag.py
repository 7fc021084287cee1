"""The fragment scan (batched, B_q <= 4, codes up to 16 words) against the
popcount scan through the C ABI. Its products are integers below 2^24 summed in
FP32 and its estimator is the popcount scan's arithmetic, so everything is
equal: integers, estimates, bounds, candidate counts, reranks and results."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# list lengths at the edges of its blocks (32 codes), code rows (64) and chunks (1024)
SIZES = [0, 1, 31, 32, 33, 63, 64, 65, 95, 127, 129, 400, 1023, 1024, 1025, 1100]


def _say(msg):
    print(f"[{msg}]", flush=True)
    sys.stdout.flush()


def _index(dim, metric=0, seed=7, bq=4, sizes=SIZES):
    import torch
    from paper_2405_12497_amd import rabitq as R
    rng = np.random.default_rng(dim * 31 + seed)
    assign = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    rng.shuffle(assign)
    cent = rng.standard_normal((len(sizes), dim)).astype(np.float32) * 0.5
    data = (cent[assign] + rng.standard_normal((len(assign), dim))).astype(np.float32)
    idx = R.Index(dim, len(sizes), seed=seed, metric=metric, bq=bq)
    idx.build(torch.from_numpy(data).cuda(), cent, assign)
    return R, idx, data, cent, rng


@pytest.mark.parametrize("words", range(1, 17))
def test_scan_export_equals_popcount(words):
    import torch
    _say(f"export {words}")
    R, idx, _, _, rng = _index(64 * words - 3)
    qu = torch.from_numpy(rng.integers(0, 16, 64 * words).astype(np.uint8)).cuda()
    for lst in (1, 2, 3, 4, 7, 12, 14):
        n = SIZES[lst]
        a = R.rbq_debug_scan(idx.h, lst, qu, 3.0, -0.07, 0.011, n, kernel=R.RBQ_SCAN_POPCNT)
        for kern in (R.RBQ_SCAN_MFMA, R.RBQ_SCAN_MFMA_FP4):
            b = R.rbq_debug_scan(idx.h, lst, qu, 3.0, -0.07, 0.011, n, kernel=kern)
            for x, y in zip(a, b):
                assert torch.equal(x, y), f"words {words} list of {n}"
    idx.close()


# rows per list around its groups of 32 queries, in every metric
@pytest.mark.parametrize("words,nq,metric", [(1, 33, 0), (2, 1, 0), (2, 130, 1), (3, 31, 2), (4, 64, 0), (5, 65, 1),
                                             (7, 32, 0), (8, 97, 2), (11, 40, 0), (12, 200, 0), (15, 33, 1), (16, 70, 0)])
def test_search_equals_popcount(words, nq, metric):
    import torch
    _say(f"search {words} {nq} {metric}")
    R, idx, data, cent, rng = _index(64 * words - 5, metric=metric)
    q = torch.from_numpy((cent[rng.integers(0, len(cent), nq)] +
                          rng.standard_normal((nq, data.shape[1]))).astype(np.float32)).cuda()
    q[0] = torch.from_numpy(data[5]).cuda()      # at distance 0 of a code
    q[-1] = torch.from_numpy(cent[4]).cuda()     # on a centroid: b = 0 for that list
    npq = torch.from_numpy(rng.integers(1, 17, nq).astype(np.int32)).cuda()
    for k, nprobe, extra in ((10, 16, {}), (1, 5, {}), (100, 16, {"nprobe_per_query": npq})):
        a = idx.search(q, k, nprobe, scan_kernel=R.RBQ_SCAN_POPCNT, stats=True, **extra)
        for kern in (R.RBQ_SCAN_MFMA, R.RBQ_SCAN_MFMA_FP4):
            b = idx.search(q, k, nprobe, scan_kernel=kern, stats=True, **extra)
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2]
    idx.close()


@pytest.mark.parametrize("dim,bq", [(700, 4), (700, 8), (1100, 4)])
def test_automatic_choice_equals_popcount(dim, bq):
    """Shapes on both sides of the automatic choice's line, host and device buffers."""
    import torch
    _say(f"automatic choice {dim} {bq}")
    rng = np.random.default_rng(3)
    R, idx, data, cent, _ = _index(dim, sizes=[70] * (1200 if bq == 4 and dim < 1000 else 300), bq=bq)
    for nq in (20, 400, 700, 1300):
        q = (cent[rng.integers(0, len(cent), nq)] + rng.standard_normal((nq, dim))).astype(np.float32)
        a = idx.search(torch.from_numpy(q).cuda(), 10, 24, scan_kernel=R.RBQ_SCAN_POPCNT, stats=True)
        b = idx.search(torch.from_numpy(q).cuda(), 10, 24, stats=True)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2]
        ids, dists, _ = idx.search(q, 10, 24)
        assert np.array_equal(ids, a[0].cpu().numpy()) and np.array_equal(dists, a[1].cpu().numpy())
        g = idx.search(torch.from_numpy(q).cuda(), 10, 24, use_graph=True)
        g = idx.search(torch.from_numpy(q).cuda(), 10, 24, use_graph=True)
        # a replay pads the batch, so an eager search of the same rows is the reference
        assert torch.equal(g[0], a[0]) and torch.equal(g[1], a[1])
    # queries that are not finite: no candidate of theirs survives, in either scan
    q = rng.standard_normal((400, dim)).astype(np.float32)
    q[3, 5] = np.nan
    q[7, 1] = np.inf
    q[9] = 1e30
    a = idx.search(torch.from_numpy(q).cuda(), 10, 24, scan_kernel=R.RBQ_SCAN_POPCNT)
    b = idx.search(torch.from_numpy(q).cuda(), 10, 24, scan_kernel=R.RBQ_SCAN_MFMA)
    assert torch.equal(a[0], b[0]) and np.array_equal(a[1].cpu().numpy(), b[1].cpu().numpy(), equal_nan=True)
    idx.close()


@pytest.mark.parametrize("words", [1, 3, 12, 16])
def test_nonfinite_base_vectors_equal_popcount(words):
    """Rows whose factors are NaN or overflow, in lists that units share with one, 31
    and 33 queries (columns without a pair repeat the last one's) and whose first
    chunk some queries scan in the bootstrap: such a row is a candidate where its
    bound compares as one and disturbs no other, so ids, distances and counts are the
    popcount scan's."""
    import torch
    from paper_2405_12497_amd import rabitq as R
    _say(f"non-finite rows {words}")
    dim, per, counts = 64 * words - 5, 1100, (1, 31, 33, 64, 2, 5)   # two chunks per list
    rng = np.random.default_rng(words)
    cent = rng.standard_normal((len(counts), dim)).astype(np.float32) * 2
    assign = np.repeat(np.arange(len(counts)), per).astype(np.int32)
    data = (cent[assign] + rng.standard_normal((len(assign), dim))).astype(np.float32)
    bad = [np.nan, np.copysign(np.nan, -1.0), np.inf, -np.inf, 1e30, -1e30, 3e38, 1e19]
    for lst in range(len(counts)):
        for i, v in enumerate(bad):   # among the first chunk's codes and the second's
            data[lst * per + 37 * i + lst] = v
            data[lst * per + 1030 + 7 * i + lst, i % dim] = v
    idx = R.Index(dim, len(counts), seed=words)
    idx.build(torch.from_numpy(data).cuda(), cent, assign)
    near = np.repeat(np.arange(len(counts)), counts)
    q = torch.from_numpy((cent[near] + rng.standard_normal((len(near), dim))).astype(np.float32)).cuda()
    many = q.repeat(16, 1)   # enough pairs for the automatic choice of wide codes
    for k, nprobe in ((10, 1), (1, 2), (100, 3), (10, 6)):
        for x, kerns in ((q, (R.RBQ_SCAN_MFMA, R.RBQ_SCAN_MFMA_FP4)), (many, (R.RBQ_SCAN_AUTO, R.RBQ_SCAN_MFMA))):
            a = idx.search(x, k, nprobe, scan_kernel=R.RBQ_SCAN_POPCNT, stats=True)
            assert torch.isfinite(a[1]).all()   # healthy rows enough for every query
            for kern in kerns:
                b = idx.search(x, k, nprobe, scan_kernel=kern, stats=True)
                assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2], (k, nprobe, kern)
    idx.close()


@pytest.mark.parametrize("dim,k,metric", [(30, 1, 0), (128, 100, 0), (255, 10, 1), (260, 33, 0), (771, 10, 2), (1027, 64, 0)])
def test_block_rerank_equals_wave_rerank(dim, k, metric):
    """A query's rerank shares by one wave each (a large batch of many lists) and
    by a block of waves each (few shares; shares of one or two lists): the rounds
    are the same, so are ids, distances and counts."""
    import torch
    _say(f"rerank {dim} {k} {metric}")
    R, idx, data, cent, rng = _index(dim, metric=metric, sizes=[40, 0, 700, 1500, 64, 3, 300, 260, 900, 128])
    q = torch.from_numpy((cent[rng.integers(0, len(cent), 400)] +
                          rng.standard_normal((400, dim))).astype(np.float32)).cuda()
    q[1] = torch.from_numpy(data[5]).cuda()
    for waves, nprobe in ((2, 10), (4, 9)):
        kw = dict(rerank_waves=waves, scan_kernel=R.RBQ_SCAN_POPCNT, stats=True)
        a = idx.search(q, k, nprobe, **kw)                # 800 or more shares of several lists
        b = idx.search(q[:100], k, nprobe, **kw)          # at most 400 shares
        assert torch.equal(a[0][:100], b[0]) and torch.equal(a[1][:100], b[1])
        c = idx.search(q, k, 2 * waves, **kw)             # shares of two lists
        d = [idx.search(q[i:i + 1], k, 2 * waves, qid_base=i, **kw) for i in range(0, 400, 16)]
        assert torch.equal(c[0][::16], torch.cat([x[0] for x in d]))
        assert torch.equal(c[1][::16], torch.cat([x[1] for x in d]))
        e = idx.search(q[:8], k, nprobe, rerank_waves=1, scan_kernel=R.RBQ_SCAN_POPCNT, stats=True)
        assert e[2]["candidates"] == idx.search(q[:8], k, nprobe, **kw)[2]["candidates"]
    idx.close()


@pytest.mark.parametrize("dim,k", [(20, 1), (64, 16), (255, 64), (300, 65), (600, 25), (1100, 100)])
def test_bootstrap_and_merge_of_small_batches(dim, k):
    """Bootstrap reranks by a block (batches up to 1024) and by a wave, and merges of
    the rerank's shares of every form (few keys; heads of up to 64 sorted lists; a
    sort), against the exact distances of the codes reranked: with a bound that
    never prunes (eps0 large) every result is the exact top k of the probed lists."""
    import torch
    _say(f"bootstrap {dim} {k}")
    R, idx, data, cent, rng = _index(dim, sizes=[300, 7, 0, 1500, 64, 3, 300, 260, 900, 128])
    R.rbq_index_set_eps0(idx.h, 200.0)
    q = (cent[rng.integers(0, len(cent), 2100)] + rng.standard_normal((2100, dim))).astype(np.float32)
    qc = torch.from_numpy(q).cuda()
    d64 = ((data[None].astype(np.float64) - q[:12, None].astype(np.float64)) ** 2).sum(-1)
    want = np.sort(d64, 1)[:, :k]
    ref = None
    for nq, waves in ((2100, 1), (2047, 1), (1025, 1), (1024, 1), (12, 1), (12, 2), (12, 40), (12, 64), (1, 64)):
        ids, d, _ = idx.search(qc[:nq], k, len(cent), rerank_waves=waves, scan_kernel=R.RBQ_SCAN_POPCNT)
        ids, d = ids[:12].cpu().numpy(), d[:12].cpu().numpy()
        ref = ref or (ids, d)
        assert np.array_equal(ids, ref[0][:nq]) and np.array_equal(d, ref[1][:nq]), (nq, waves)
    # FP32 sums of dim terms: relative error below (dim / 8 + 8) 2^-23
    assert (np.abs(ref[1] - want) <= want * (dim / 8 + 8) * 2.0 ** -23 + 1e-12).all()
    idx.close()


@pytest.mark.parametrize("nprobe", [1, 7, 10])
def test_batches_around_the_plan(nprobe):
    """Batches planned by one launch (4 queries), scanned by one block (1024) and by
    several: a query's results and the counts do not depend on the batch."""
    import torch
    _say(f"plan {nprobe}")
    R, idx, data, cent, rng = _index(40, sizes=[300, 7, 0, 1500, 64, 3, 300, 260, 900, 128])
    q = torch.from_numpy((cent[rng.integers(0, len(cent), 2050)] +
                          rng.standard_normal((2050, 40))).astype(np.float32)).cuda()
    kw = dict(rerank_waves=1, scan_kernel=R.RBQ_SCAN_POPCNT)
    ref = idx.search(q, 10, nprobe, **kw)
    for nq in (1, 3, 4, 5, 64, 1023, 1024, 1025, 2048, 2049):
        a = idx.search(q[:nq], 10, nprobe, stats=True, **kw)
        assert torch.equal(a[0], ref[0][:nq]) and torch.equal(a[1], ref[1][:nq]), nq
        b = idx.search(q[:nq], 10, nprobe, rerank_waves=1, scan_kernel=R.RBQ_SCAN_MFMA, stats=True)
        assert torch.equal(a[0], b[0]) and a[2] == b[2], nq
    idx.close()


@pytest.mark.parametrize("words", range(5, 17))
def test_wide_pair_quantisation(words):
    """4-bit rounding of 5 to 16 words against its definition, floor((r - min) / step
    + u) with the counter stream's u: equal wherever that argument is at least 1e-3
    from an integer (FP32 steps of 15 levels are good to 1e-5), one level off at most
    elsewhere. Seeds with and without carries that differ inside a draw; batches of
    few pairs and of several pairs per wave; empty and NaN residuals."""
    import torch
    from oracle import rabitq_oracle as O
    from paper_2405_12497_amd import rabitq as R
    _say(f"pair quantisation {words}")
    dim, dp, nlist = 64 * words - 9, 64 * words, 40
    for seed in (7, 960):
        rng = np.random.default_rng(words)
        P = np.linalg.qr(rng.standard_normal((dp, dp)))[0]
        cent = rng.standard_normal((nlist, dim)).astype(np.float32)
        data = rng.standard_normal((200, dim)).astype(np.float32)
        idx = R.Index(dim, nlist, seed=seed)
        idx.build_rotation(data, cent, (np.arange(200) % nlist).astype(np.int32), P)
        crot = (cent.astype(np.float64) @ P[:dim]).astype(np.float32)
        for nq, nprobe, base in ((3, 5, 0), (2600, 33, 1000)):
            q = rng.standard_normal((nq, dim)).astype(np.float32)
            q[1] = cent[3]                 # a residual of rounding errors only
            q[2, 5] = np.nan
            lists = np.stack([rng.permutation(nlist)[:nprobe] for _ in range(nq)]).astype(np.int32)
            qc = torch.from_numpy(q).cuda()
            qu, scal = R.rbq_debug_quantize(idx.h, qc, torch.from_numpy(lists).cuda(), dp, qid_base=base)
            qu, scal = qu.cpu().numpy().reshape(nq, nprobe, dp), scal.cpu().numpy().reshape(nq, nprobe, 4)
            rot = R.rbq_debug_rotate(idx.h, qc, dp).cpu().numpy()
            assert (qu[2] == 0).all()      # NaN quantises to 0
            near = total = 0
            for qi in [0] + list(range(3, nq, 97)):
                for r in range(0, nprobe, 1 if nq < 10 else 4):
                    lid = int(lists[qi, r])
                    res = (rot[qi] - crot[lid]).astype(np.float64)
                    step = (res.max() - res.min()) / 15
                    v = (res - res.min()) / step + O.rounding_uniforms_fast(seed, base + qi, lid, dp)
                    clear = np.abs(v - np.rint(v)) > 1e-3
                    want = np.clip(np.floor(v), 0, 15)
                    assert (qu[qi, r][clear] == want[clear]).all(), (seed, qi, r)
                    assert (np.abs(qu[qi, r] - want) <= 1).all()
                    b = np.linalg.norm(res)     # v_l and the step are of the unit residual
                    assert abs(scal[qi, r, 1] * b - res.min()) <= 1e-5 * np.abs(res).max()
                    assert abs(scal[qi, r, 2] * b - step) <= 1e-5 * step
                    assert scal[qi, r, 3] == qu[qi, r].sum()
                    near += int((~clear).sum())
                    total += dp
            assert near <= 0.01 * total
        idx.close()


@pytest.mark.parametrize("words,seed", [(5, 7), (8, 960), (12, 7), (12, 960), (16, 7), (15, 960)])
def test_search_quantises_as_the_export(words, seed):
    """What a search writes of a pair (bit planes; the fragment scan's rows) holds the
    exported rounding: one list of two chunks and a part, the first the bootstrap's.
    The candidates counted are that chunk's codes and the later ones whose exported
    bound is at most the k-th exact distance of the 4k best exported estimates. FP32
    sums and the export's FP32 scalars: codes within 1e-5 of the distances' scale of
    that threshold may count either way."""
    import torch
    from paper_2405_12497_amd import rabitq as R
    _say(f"search rounding {words} {seed}")
    dim, n, k, nq, base = 64 * words - 9, 2500, 10, 24, 50
    rng = np.random.default_rng(words)
    cent = rng.standard_normal((1, dim)).astype(np.float32)
    data = (cent + rng.standard_normal((n, dim))).astype(np.float32)
    q = (cent + rng.standard_normal((nq, dim))).astype(np.float32)
    idx = R.Index(dim, 1, seed=seed)
    idx.build(data, cent, np.zeros(n, np.int32))
    qc = torch.from_numpy(q).cuda()
    order = R.rbq_debug_list_ids(idx.h, 0, n)
    one = torch.zeros((nq, 1), dtype=torch.int32, device="cuda")

    def bounds(first_id):
        """Fewest and most candidates of each query, rounded as ids first_id, ... are."""
        qu, scal = R.rbq_debug_quantize(idx.h, qc, one, 64 * words, qid_base=first_id)
        scal = scal.cpu().numpy()
        lo, hi = [], []
        for i in range(nq):
            _, _, _, dist, lb = R.rbq_debug_scan(idx.h, 0, qu[i], *map(float, scal[i, :3]), n)
            dist, lb = dist.cpu().numpy()[:1024], lb.cpu().numpy().astype(np.float64)
            d = ((data[order].astype(np.float64) - q[i]) ** 2).sum(1)
            best = np.argsort(dist, kind="stable")
            eps = 1e-5 * d.mean()
            taus = [np.sort(d[best[:m]])[k - 1] for m in (4 * k - 1, 4 * k, 4 * k + 1)]   # equal estimates at the cut
            lo.append(1024 + int((lb[1024:] <= min(taus) - eps).sum()))
            hi.append(1024 + int((lb[1024:] <= max(taus) + eps).sum()))
        return np.array(lo), np.array(hi)

    lo, hi = bounds(base)
    share = (lo - 1024) / (n - 1024)
    assert 0.02 < share.mean() < 0.8 and (hi - lo).mean() < 10
    other = bounds(base + 1000)[0]   # another rounding of the same queries: the counts tell them apart
    assert (np.abs(other - lo) > hi - lo).mean() > 0.5
    for kern in (R.RBQ_SCAN_POPCNT, R.RBQ_SCAN_MFMA):
        got = np.array([idx.search(qc[i:i + 1], k, 1, qid_base=base + i, scan_kernel=kern, rerank_waves=1,
                                   stats=True)[2]["candidates"] for i in range(nq)])
        assert ((lo <= got) & (got <= hi)).all(), (kern, lo, got, hi)
    idx.close()
