"""The one-workgroup-per-query way of a search against the general way (list sharing mode 0) and float64: same short-lists,
same results, bit for bit, over the forms that it takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _index(rng, d, c, m, lengths, mr=8, distinct=256):
    import paper_1102_3828_amd as pkg
    N = int(sum(lengths))
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    coarse = rng.uniform(0, 100, (c, d)).astype(np.float32)
    pq = rng.normal(0, 15, (m, 256, d // m)).astype(np.float32)
    rq = rng.normal(0, 8, (mr, 256, d // mr)).astype(np.float32) if mr else None
    codes = rng.integers(0, distinct, (N, m)).astype(np.uint8)
    rcodes = rng.integers(0, 256, (N, mr)).astype(np.uint8) if mr else None
    ids = rng.permutation(N).astype(np.int32)
    ix = pkg.Index(d, c, m, mr)
    ix.set_codebooks(coarse, pq, rq)
    ix.import_(offsets, ids, codes, rcodes)
    return ix, dict(coarse=coarse, pq=pq, codes=codes, ids=ids, offsets=offsets)


def _by_query(ix):
    """Whether the last search ran one workgroup per query (set_profiling(2)): that way has no sample."""
    t = ix.stage_times()
    return t["scan"] > 0 and t["sample"] == 0


def _both(ix, x, w, kp, k, table_mode, by_query=True, left_out=False):
    """The call left to itself, which must go the way that is asked for, and sharing mode 0: the same in every bit.  left_out: the
    first leaves lists out, of at least half of the entries."""
    import torch
    xq = torch.from_numpy(x).cuda()
    ix.set_table_mode(table_mode)
    ix.set_profiling(2)
    out = []
    for mode in (-1, 0):
        ix.set_list_sharing(mode)
        ids, dist, t = ix.search(xq, w, kp, k, trace=True)
        assert _by_query(ix) == (by_query and mode == -1), (len(x), w, kp)
        st = ix.search_stats()
        if mode == -1 and left_out:
            assert 0 < st["codes_streamed"] < 0.5 * st["codes_scanned"]
        else:
            assert st["codes_streamed"] <= st["codes_scanned"] and (mode == -1 or st["codes_streamed"] == st["codes_scanned"])
        ids2, dist2 = ix.search(xq, w, kp, k)
        assert torch.equal(ids, ids2) and torch.equal(dist, dist2)
        n = t["short_count"].cpu().numpy()
        s_ids, s_est = t["short_ids"].cpu().numpy(), t["short_est"].cpu().numpy()
        filled = np.arange(kp)[None, :] < n[:, None]
        order = np.lexsort((s_ids, np.where(filled, s_est, np.inf)))
        short = [np.take_along_axis(np.where(filled, v, 0), order, 1) for v in (s_ids, s_est)]
        out.append((ids.cpu().numpy(), dist.cpu().numpy(), n, *short, t["probe"].cpu().numpy(),
                    np.array([st["codes_scanned"], st["pairs"]])))
    for a, b in zip(*out):
        assert (a == b).all()
    return out[0]


@pytest.mark.parametrize("table_mode", [0, 1])
@pytest.mark.parametrize("m", [4, 8, 16, 32, 64])
def test_same_results_as_the_general_way(m, table_mode):
    """Short lists, empty ones among them: several lists' tables in LDS at a time, entries kept in visit order.  200 queries
    have a compute unit each, 300 share them (not with m = 64)."""
    rng = np.random.default_rng(m)
    c = 40
    lengths = rng.integers(0, 1200, c)
    lengths[[3, 4, 20]] = 0                       # lists without an entry
    lengths[7], lengths[8], lengths[9] = 1, 1023, 1025
    ix, _ = _index(rng, 64, c, m, lengths)
    x = rng.uniform(0, 100, (300, 64)).astype(np.float32)
    for w, kp, k in ((1, 1, 1), (1, 1000, 10), (5, 512, 512), (5, 513, 20), (8, 100, 100), (8, 1024, 300), (20, 512, 9), (20, 1000, 1000)):
        if (w > 8 and m > 8) or (w > 5 and m > 32):
            continue
        _both(ix, x[:200], w, kp, k, table_mode)
        _both(ix, x, w, kp, k, table_mode, by_query=m < 64)
        if w < (5 if m > 16 else 8):
            _both(ix, x[:9], w, kp, k, table_mode)
    _both(ix, x[:200], 5, 1025, 10, table_mode, by_query=False)


@pytest.mark.parametrize("table_mode", [0, 1])
@pytest.mark.parametrize("m", [4, 8, 16, 32, 64])
def test_long_visits_are_cut_to_the_short_list_as_they_go(m, table_mode):
    """Visits around and beyond the places (16384 entries of a query that has a compute unit to itself, 8192 of one that shares
    it): the bare estimates of a visit that fits, records that are cut to the k' best whenever the places run out."""
    rng = np.random.default_rng(m + 50)
    lengths = np.array([10000, 9500, 6500, 6000, 5000, 5500, 0, 1])
    ix, _ = _index(rng, 64, 8, m, lengths)
    x = rng.uniform(0, 100, (300, 64)).astype(np.float32)
    for w in (2, 3, 8):
        if (w > 2 and m > 32) or (w > 3 and m > 16):
            continue
        for kp, k in ((1, 1), (100, 100), (512, 30), (513, 513), (1024, 1000)):
            for nq, places in ((250, 16384), (300, 8192)):
                if nq > 256 and m > 32:
                    continue
                probe = _both(ix, x[:nq], w, kp, k, table_mode)[5]
                visits = lengths[probe].sum(1)
                assert visits.max() > places and (w > 3 or visits.min() <= places)
        if w == 2:     # three queries: wide codes are spread over the chip
            if m != 16:
                _both(ix, x[:3], w, 100, 10, table_mode, by_query=m < 16)


def test_short_list_against_float64():
    rng = np.random.default_rng(11)
    ix, b = _index(rng, 64, 16, 8, rng.integers(500, 3000, 16))
    x = rng.uniform(0, 100, (200, 64)).astype(np.float32)
    for w, kp in ((3, 700), (16, 700), (16, 3)):
        _, _, n, s_ids, *_ = _both(ix, x, w, kp, 1, 0)
        for q in range(0, len(x), 33):
            dc = ((x[q].astype(np.float64) - b["coarse"]) ** 2).sum(1)
            est = []
            for l in np.argsort(dc)[:w]:
                r = (x[q].astype(np.float64) - b["coarse"][l]).reshape(8, 1, 8)
                tab = ((r - b["pq"].astype(np.float64)) ** 2).sum(-1)
                a, e = b["offsets"][l], b["offsets"][l + 1]
                est += list(zip(tab[np.arange(8), b["codes"][a:e]].sum(1), b["ids"][a:e]))
            est.sort()
            want = {i for _, i in est[:kp]}
            edge = est[kp - 1][0]
            by_id = {i: v for v, i in est}
            got = set(s_ids[q, :n[q]])
            # what differs must sit on the edge: 8 table entries and 7 additions, each within a few ulp of the largest term
            assert n[q] == kp and all(abs(by_id[i] - edge) <= 2e-6 * edge for i in got ^ want)


@pytest.mark.parametrize("distinct", [1, 2])
def test_crowds_of_equal_estimates_are_cut_by_id(distinct):
    """Every code the same, or two per sub-quantizer: thousands of entries share the k'-th estimate, in visits that fit the
    places and in visits that are cut more than once."""
    rng = np.random.default_rng(distinct)
    ix, _ = _index(rng, 64, 6, 4, [9000, 3000, 5000, 100, 0, 7000], distinct=distinct)
    x = rng.uniform(0, 100, (300, 64)).astype(np.float32)
    for w, kp, k in ((1, 300, 7), (6, 300, 300), (6, 1000, 40), (6, 1024, 10)):
        _both(ix, x[:250], w, kp, k, 0)
        _both(ix, x, w, kp, k, 0)


@pytest.mark.parametrize("kp", [100, 500, 1000])
def test_entries_that_get_better_and_better(kp):
    """Inside every list the estimates fall from entry to entry: each pass beats the bound of the one before."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(kp)
    c, d, n = 3, 32, 12000
    coarse = np.zeros((c, d), dtype=np.float32)
    pq = np.zeros((4, 256, 8), dtype=np.float32)
    pq[:, :, 0] = np.arange(256)[None, :]
    lists = []
    for l in range(c):
        v = np.sort(rng.integers(0, 256 ** 2, n))[::-1]
        lists.append(np.stack([v >> 8, v >> 8, v & 255, v & 255], axis=1).astype(np.uint8))
    codes = np.concatenate(lists)
    ix = pkg.Index(d, c, 4, 0)
    ix.set_codebooks(coarse, pq)
    ix.import_(np.arange(c + 1) * n, rng.permutation(c * n).astype(np.int32), codes)
    x = rng.uniform(0, 3, (300, d)).astype(np.float32)
    _both(ix, x[:250], 3, kp, 50, 0)
    _both(ix, x, 3, kp, 50, 0)


def test_ids_that_repeat_stay_inside_the_places():
    """Every entry has the same key (repeated ids are not allowed, but nothing checks them): each cut to the k' best keeps k'
    records although all of them lie at or below the pivot, and the next ones must follow those."""
    import torch
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(2)
    d, n, nq, kp = 32, 40000, 250, 100
    coarse = rng.uniform(0, 100, (2, d)).astype(np.float32)
    pq = rng.normal(0, 15, (4, 256, d // 4)).astype(np.float32)
    ix = pkg.Index(d, 2, 4, 0)
    ix.set_codebooks(coarse, pq)
    ix.import_([0, n, 2 * n], np.full(2 * n, 7, np.int32), np.full((2 * n, 4), 3, np.uint8))
    ix.set_profiling(2)
    x = rng.uniform(0, 100, (nq, d)).astype(np.float32)
    ids, dist, t = ix.search(torch.from_numpy(x).cuda(), 1, kp, 10, trace=True)
    assert _by_query(ix)
    near = ((x[:, None, :].astype(np.float64) - coarse) ** 2).sum(-1).argmin(1)
    want = ((x.astype(np.float64) - coarse[near] - pq[:, 3].reshape(-1)) ** 2).sum(1)
    assert (t["short_count"] == kp).all() and (t["short_ids"] == 7).all() and (ids == 7).all()
    # 32 squares of differences around 20 between values up to 160: 2 * 160 / 20 + 2 half-ulps each, 8 for the additions
    assert (np.abs(dist.cpu().numpy() / want[:, None] - 1) < 26 * 2.0 ** -24).all()


def test_many_visited_lists_and_many_queries():
    rng = np.random.default_rng(5)
    ix, _ = _index(rng, 32, 600, 4, rng.integers(0, 60, 600), mr=4)
    x = rng.uniform(0, 100, (300, 32)).astype(np.float32)
    for w in (1, 63, 64, 65, 128, 150):
        _both(ix, x, w, 200, 20, 0)
    _both(ix, x, 512, 200, 20, 0, by_query=False)


def test_fixed_workspace():
    """search_static takes the same way (it times nothing, so this asserts the results only)."""
    import torch
    rng = np.random.default_rng(6)
    ix, _ = _index(rng, 64, 8, 8, [10000, 9500, 6500, 6000, 5000, 5500, 0, 1])
    x = rng.uniform(0, 100, (300, 64)).astype(np.float32)
    for nq, w, kp, k in ((1, 1, 100, 10), (250, 3, 1000, 257), (300, 8, 500, 50)):
        want = _both(ix, x[:nq], w, kp, k, 0)
        ix.set_list_sharing(-1)
        ids = torch.empty((nq, k), dtype=torch.int32, device="cuda")
        dist = torch.empty((nq, k), dtype=torch.float32, device="cuda")
        ix.search_static(torch.from_numpy(x[:nq]).cuda(), w, kp, k, ids, dist)
        assert (ids.cpu().numpy() == want[0]).all() and (dist.cpu().numpy() == want[1]).all()


@pytest.mark.parametrize("d", [16, 64])
@pytest.mark.parametrize("mode", [-1, 0])
def test_the_last_query_that_is_not_finite_is_named(d, mode):
    """Several in a batch, in different workgroups of the distance kernel: the same one is named whichever way the call goes and
    whichever writes first; the next call is not affected."""
    import torch
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(d)
    ix, _ = _index(rng, d, 8, 4, [300] * 8, mr=0)
    ix.set_profiling(2)
    ix.set_list_sharing(mode)
    x = rng.uniform(0, 100, (400, d)).astype(np.float32)
    good = torch.from_numpy(x).cuda()
    want = ix.search(good, 2, 50, 5)
    assert _by_query(ix) == (mode == -1)
    for rows in ([0, 64, 130, 131, 398], [399], [5, 3], [63, 64]):
        bad = x.copy()
        for i, r in enumerate(rows):
            bad[r, i % d] = (np.nan, np.inf, -np.inf, 3e19)[i % 4]
        with pytest.raises(pkg.IvfrError) as e:
            ix.search(torch.from_numpy(bad).cuda(), 2, 50, 5)
        assert e.value.code == pkg.binding.ERR_INVALID_ARG and f"query {max(rows)} " in str(e.value)
        got = ix.search(good, 2, 50, 5)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("m,ds", [(4, 8), (4, 32), (8, 8), (8, 16), (8, 32), (16, 8), (16, 16)])
@pytest.mark.parametrize("kp", [40, 700])
def test_lists_beyond_the_short_list_are_left_out(m, ds, kp):
    """Queries near a centroid, the other lists far away.  Visits that fit, too few entries in the near lists for a bound, lists that
    are all empty but the last, and visits that do not fit, of which most is left out."""
    rng = np.random.default_rng(m * ds + kp)
    c, w, d = 48, 12, m * ds
    lengths = rng.integers(300, 700, c)
    lengths[[3, 4, 20, 21]] = 0
    lengths[10] = 5000
    ix, s = _index(rng, d, c, m, lengths)
    near = s["coarse"][rng.integers(0, c, 280)] + rng.normal(0, 15, (280, d))
    x = np.concatenate([near, rng.uniform(0, 100, (20, d))]).astype(np.float32)
    for visit in (2, 6, w):
        if m * visit <= 128:
            _both(ix, x, visit, kp, 30, 0)
    lengths = np.zeros(c, int)
    lengths[:9] = 900
    ix, s = _index(rng, d, c, m, lengths)
    if m <= 8:
        _both(ix, (s["coarse"][rng.integers(0, c, 300)] + rng.normal(0, 3, (300, d))).astype(np.float32), w, kp, 30, 0)
    # visits that do not fit: the first cut is a bound that only the nearest lists reach, the others are not read
    ix, s = _index(rng, d, c, m, rng.integers(1200, 1800, c))
    near = s["coarse"][rng.integers(0, c, 280)] + rng.normal(0, 15, (280, d))
    _both(ix, near.astype(np.float32), 30 if m == 4 else w, kp, 30, 0, left_out=True)
