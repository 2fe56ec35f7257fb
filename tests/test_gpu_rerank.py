"""Re-rank (Eq. (9)-(10)) of every shape its kernels distinguish, against float64 on the same codes, through the C ABI."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# relative error of a distance: every term carries the rounding of three differences, a chain adds 16 terms and the chains
# are combined in at most four steps: (2 * 3 + 16 + 4) half-ulps of 2^-24
REL = 26 * 2.0 ** -24


def _index(rng, d, c, m, mr, N):
    import paper_1102_3828_amd as pkg
    coarse = rng.uniform(0, 100, (c, d)).astype(np.float32)
    pq = rng.normal(0, 15, (m, 256, d // m)).astype(np.float32)
    rq = rng.normal(0, 8, (mr, 256, d // mr)).astype(np.float32) if mr else None
    lists = np.sort(rng.integers(0, c, N))
    offsets = np.zeros(c + 1, dtype=np.int64)
    np.cumsum(np.bincount(lists, minlength=c), out=offsets[1:])
    ids = rng.permutation(N).astype(np.int32)
    codes = rng.integers(0, 256, (N, m)).astype(np.uint8)
    rcodes = rng.integers(0, 256, (N, mr)).astype(np.uint8)
    ix = pkg.Index(d, c, m, mr)
    ix.set_codebooks(coarse, pq, rq)
    ix.import_(offsets, ids, codes, rcodes if mr else None)
    y = coarse.astype(np.float64)[lists] + pq.astype(np.float64)[np.arange(m), codes].reshape(N, d)
    if mr:
        y += rq.astype(np.float64)[np.arange(mr), rcodes].reshape(N, d)
    by_id = np.empty_like(y)
    by_id[ids] = y
    return ix, by_id


@pytest.mark.parametrize("d,m,mr", [(64, 4, 0), (64, 8, 16), (64, 16, 4), (128, 4, 8), (128, 8, 0), (128, 8, 16), (128, 16, 32),
                                    (128, 32, 4), (256, 8, 64), (256, 64, 8), (256, 16, 16), (128, 64, 8), (32, 8, 4), (512, 16, 16),
                                    (32, 4, 0), (32, 4, 4), (32, 4, 8), (32, 8, 8), (32, 8, 16)])
def test_refined_distances_of_every_shape(d, m, mr):
    import torch
    rng = np.random.default_rng(d * 1000 + m * 10 + mr)
    ix, y = _index(rng, d, 24, m, mr, 6000)
    x = rng.uniform(0, 100, (5, d)).astype(np.float32)
    xq = torch.from_numpy(x).cuda()
    # short-lists around the rounds of a workgroup, shorter and longer than what is visited, few and many results
    for w, kp, k in ((24, 1, 1), (24, 127, 5), (24, 129, 129), (3, 256, 256), (24, 300, 257), (24, 512, 10), (24, 513, 513),
                     (24, 1024, 256), (24, 1025, 100), (24, 2600, 7), (2, 4000, 300), (24, 6000, 3000)):
        ids, dist, t = ix.search(xq, w, kp, k, trace=True)
        ids2, dist2 = ix.search(xq, w, kp, k)
        assert torch.equal(ids, ids2) and torch.equal(dist, dist2)
        ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
        n_short = t["short_count"].cpu().numpy()
        s_ids, s_ref = t["short_ids"].cpu().numpy(), t["short_ref"].cpu().numpy()
        for q in range(len(x)):
            n = n_short[q]
            assert (s_ids[q, n:] == -1).all() and np.isinf(s_ref[q, n:]).all()
            ref = ((x[q].astype(np.float64) - y[s_ids[q, :n]]) ** 2).sum(1)
            assert (np.abs(s_ref[q, :n] - ref) <= REL * ref).all(), (w, kp, k, q, np.abs(s_ref[q, :n] / ref - 1).max())
            order = np.lexsort((s_ids[q, :n], s_ref[q, :n]))[:k]
            n_out = min(k, n)
            assert (ids[q, :n_out] == s_ids[q, :n][order]).all() and (dist[q, :n_out] == s_ref[q, :n][order]).all()
            assert (ids[q, n_out:] == -1).all() and np.isinf(dist[q, n_out:]).all()


@pytest.mark.parametrize("d,m,mr", [(32, 4, 8), (32, 8, 8), (64, 8, 16), (128, 4, 0), (128, 8, 32), (256, 16, 8)])
def test_many_queries_and_few_give_the_same_bits(d, m, mr):
    """Few entries are decoded one round of 128 per workgroup, many in as many rounds as a short-list needs (more than 65536
    entries on 256 compute units): every entry's sum is the same, whichever workgroup has it."""
    import torch
    rng = np.random.default_rng(d + m)
    ix, _ = _index(rng, d, 24, m, mr, 6000)
    # one, two, four and eight rounds; the k best inside and outside; several workgroups per query
    for kp, k in ((128, 128), (129, 5), (257, 257), (512, 30), (513, 256), (1024, 300), (1025, 40), (4000, 9)):
        nq = 65536 // kp + 5
        xq = torch.from_numpy(rng.uniform(0, 100, (nq, d)).astype(np.float32)).cuda()
        ids, dist, t = ix.search(xq, 24, kp, k, trace=True)
        ids2, dist2 = ix.search(xq, 24, kp, k)
        assert torch.equal(ids, ids2) and torch.equal(dist, dist2)
        for a in (0, nq // 2, nq - 4):
            few_ids, few_dist, few = ix.search(xq[a:a + 4].contiguous(), 24, kp, k, trace=True)
            assert torch.equal(few_ids, ids[a:a + 4]) and torch.equal(few_dist, dist[a:a + 4])
            for q in range(4):
                both = [dict(zip(u["short_ids"][i].tolist(), u["short_ref"][i].tolist())) for u, i in ((few, q), (t, a + q))]
                assert both[0] == both[1]


@pytest.mark.parametrize("c,w", [(200, 128), (200, 129), (16384, 128), (20000, 60)])
def test_refined_distances_with_many_visited_lists(c, w):
    """Residuals in LDS up to 128 visited lists of at most 16384; centroids from memory beyond."""
    import torch
    rng = np.random.default_rng(c + w)
    ix, y = _index(rng, 64, c, 8, 8, 40000)
    x = rng.uniform(0, 100, (4, 64)).astype(np.float32)
    ids, dist, t = ix.search(torch.from_numpy(x).cuda(), w, 700, 50, trace=True)
    s_ids, s_ref, n_short = (t[k].cpu().numpy() for k in ("short_ids", "short_ref", "short_count"))
    for q in range(4):
        n = n_short[q]
        ref = ((x[q].astype(np.float64) - y[s_ids[q, :n]]) ** 2).sum(1)
        assert n > 50 and (np.abs(s_ref[q, :n] - ref) <= REL * ref).all()
        order = np.lexsort((s_ids[q, :n], s_ref[q, :n]))[:50]
        assert (ids.cpu().numpy()[q] == s_ids[q, :n][order]).all()


@pytest.mark.parametrize("c,d", [((1 << 20) + 5, 64), ((1 << 22) + 9, 128)])
def test_refined_distances_with_centroids_beyond_2_to_31_bytes(c, d):
    """More than 2^20 lists; centroid rows on both sides of byte 2^31."""
    import torch
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(c)
    near = np.unique(np.concatenate([[0, c - 1, c // 2, c // 2 + 1], rng.integers(0, c, 40)]))   # the others lie far off
    coarse = np.full((c, d), 1000.0, dtype=np.float32)
    coarse[near] = rng.uniform(0, 100, (len(near), d))
    pq = rng.normal(0, 15, (8, 256, d // 8)).astype(np.float32)
    rq = rng.normal(0, 8, (8, 256, d // 8)).astype(np.float32)
    N = 9000
    lists = np.sort(rng.choice(near, N))
    offsets = np.searchsorted(lists, np.arange(c + 1)).astype(np.int64)
    codes, rcodes = rng.integers(0, 256, (2, N, 8)).astype(np.uint8)
    ix = pkg.Index(d, c, 8, 8)
    ix.set_codebooks(coarse, pq, rq)
    ix.import_(offsets, np.arange(N, dtype=np.int32), codes, rcodes)
    y = coarse[lists].astype(np.float64) + (pq[np.arange(8), codes].astype(np.float64) + rq[np.arange(8), rcodes]).reshape(N, d)
    x = rng.uniform(0, 100, (70, d)).astype(np.float32)
    for nq in (3, 70):       # one round per workgroup, eight
        _, _, t = ix.search(torch.from_numpy(x[:nq]).cuda(), len(near), 1000, 10, trace=True)
        s_ids, s_ref = t["short_ids"].cpu().numpy(), t["short_ref"].cpu().numpy()
        assert (t["short_count"] == 1000).all()
        for q in range(nq):
            ref = ((x[q].astype(np.float64) - y[s_ids[q]]) ** 2).sum(1)
            assert (np.abs(s_ref[q] - ref) <= REL * ref).all()


@pytest.mark.parametrize("values", [1, 3, 256])
def test_sorted_results_of_every_length(values):
    """Counting, bins and network: as many results as each takes, with crowds of equal distances and without."""
    import torch
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(values)
    N, c, d, m = 12000, 4, 64, 8
    offsets = np.array([0, 5000, 5000, 9000, N])
    codes = np.repeat(rng.integers(0, values, (N, 1)), m, axis=1).astype(np.uint8) if values < 256 else rng.integers(0, 256, (N, m)).astype(np.uint8)
    ids = rng.permutation(N).astype(np.int32)
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(rng.uniform(0, 100, (c, d)), rng.normal(0, 9, (m, 256, 8)))
    ix.import_(offsets, ids, codes)
    x = torch.from_numpy(rng.uniform(0, 100, (3, d)).astype(np.float32)).cuda()
    for kp, k in ((12000, 257), (12000, 512), (12000, 513), (6000, 4096), (12000, 5000), (8000, 8000), (12000, 8192), (12000, 8193), (12000, 12000), (13000, 13000)):
        ids_o, dist, t = ix.search(x, c, kp, k, trace=True)
        s_ids, s_ref = t["short_ids"].cpu().numpy(), t["short_ref"].cpu().numpy()
        for q in range(3):
            n = int(t["short_count"][q])
            order = np.lexsort((s_ids[q, :n], s_ref[q, :n]))[:k]
            assert n == min(kp, N)
            assert (ids_o[q, :len(order)].cpu().numpy() == s_ids[q, order]).all() and (dist[q, :len(order)].cpu().numpy() == s_ref[q, order]).all()
            assert (ids_o[q, len(order):] == -1).all()


@pytest.mark.parametrize("d,m,nq,w", [(64, 64, 3, 5), (64, 32, 1, 1), (64, 16, 40, 7), (128, 64, 2, 9), (256, 64, 5, 3)])
def test_tables_of_narrow_sub_vectors(d, m, nq, w):
    """Eq. (5) with 1, 2 and 4 dimensions per sub-quantizer, pairs that do not fill a workgroup: estimates against float64."""
    import torch
    rng = np.random.default_rng(d + m)
    ix, _ = _index(rng, d, 12, m, 0, 900)
    ix.set_list_sharing(0)        # tables from memory
    coarse, pq, _ = ix.get_codebooks()
    offsets, ids, codes, _ = ix.export()
    x = rng.uniform(0, 100, (nq, d)).astype(np.float32)
    _, _, t = ix.search(torch.from_numpy(x).cuda(), w, 2000, 1, trace=True)
    entry = np.argsort(ids)
    lists = np.repeat(np.arange(12), np.diff(offsets))
    for q in range(nq):
        n = int(t["short_count"][q])
        e = entry[t["short_ids"][q, :n].cpu().numpy()]
        y = coarse.astype(np.float64)[lists[e]] + pq.astype(np.float64)[np.arange(m), codes[e]].reshape(n, d)
        est = ((x[q].astype(np.float64) - y) ** 2).sum(1)
        # m table entries of d / m squares each, then m additions in two chains
        assert (np.abs(t["short_est"][q, :n].cpu().numpy() - est) <= (m / 2 + d / m + 6) * 2.0 ** -24 * est).all()
