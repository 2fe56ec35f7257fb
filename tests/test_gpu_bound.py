"""Lists left out because their smallest possible estimate lies above a query's bound: the call left to itself against every
pair scanned on its own (sharing mode 0), bit for bit, short-lists included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _index(rng, d, c, m, n, codes):
    import paper_1102_3828_amd as pkg
    coarse = rng.uniform(0, 100, (c, d)).astype(np.float32)
    pq = rng.normal(0, 12, (m, 256, d // m)).astype(np.float32)
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, pq, None)
    ix.import_(np.arange(c + 1, dtype=np.int64) * n, rng.permutation(c * n).astype(np.int32), codes)
    return ix, coarse, pq


def _run(ix, x, w, kp, k, mode):
    import torch
    ix.set_list_sharing(mode)
    ids, dist, t = ix.search(torch.from_numpy(x).cuda(), w, kp, k, trace=True)
    n = t["short_count"].cpu().numpy()
    s_ids, s_est = t["short_ids"].cpu().numpy(), t["short_est"].cpu().numpy()
    short = [sorted(zip(s_est[q, :n[q]].tolist(), s_ids[q, :n[q]].tolist())) for q in range(len(x))]
    return (ids.cpu().numpy(), dist.cpu().numpy(), n, short), ix.search_stats()


def _same(a, b):
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and (a[2] == b[2]).all() and a[3] == b[3]


@pytest.mark.parametrize("m,ds", [(4, 8), (4, 16), (4, 32), (8, 8), (8, 16), (8, 32), (16, 8), (16, 16)])
def test_lists_beyond_the_bound_are_left_out(m, ds):
    rng = np.random.default_rng(100 * m + ds)
    d, c, n, w = m * ds, 12, 25001, 7
    ix, coarse, _ = _index(rng, d, c, m, n, rng.integers(0, 256, (c * n, m)).astype(np.uint8))
    # near a centroid (the other lists hold nothing), between the centroids, and far from all of them; pairs that do not fill the
    # last wavefront
    x = np.concatenate([coarse[rng.integers(0, c, 1500)] + rng.normal(0, 12, (1500, d)), rng.uniform(0, 100, (500, d)),
                        rng.uniform(-3000, 3000, (3, d))]).astype(np.float32)
    kp = 60
    shared, st2 = _run(ix, x, w, kp, 10, 2)
    left, st = _run(ix, x, w, kp, 10, -1)
    alone, _ = _run(ix, x, w, kp, 10, 0)
    _same(left, alone)
    _same(left, shared)
    assert st["dense_fallbacks"] == st["bound_retries"] == 0 and st["codes_scanned"] == st2["codes_scanned"] == len(x) * w * n >= 3e8
    # about two thirds of the work is left out (31 to 36 % is done over these shapes), and the rest does not move to single pairs
    parts = ("codes_scanned_shared", "codes_scanned_shared2", "codes_scanned_shared8")
    assert sum(st[p] for p in parts) < 0.4 * sum(st2[p] for p in parts) and st["codes_streamed"] < 0.4 * st2["codes_streamed"]


@pytest.mark.parametrize("c,w,big", [(1, 1, 2), (63, 9, 2), (1024, 16, 2), (1025, 16, 3), (8192, 8, 2), (8193, 70, 2), (20000, 16, 3)])
def test_grouping_of_the_pairs_by_list(c, w, big):
    """One list a lane, eight, and a second step over the lists; one and more than one step of the plan over a query's pairs; units of
    every size, those of 64 among them (mode 3): every pair is scanned once, whichever unit has it."""
    rng = np.random.default_rng(c + w)
    ix, coarse, _ = _index(rng, 32, c, 4, 40, rng.integers(0, 256, (c * 40, 4)).astype(np.uint8))
    x = (coarse[rng.integers(0, c, 900) % 40] + rng.normal(0, 12, (900, 32))).astype(np.float32)   # some lists often, most never
    shared, st = _run(ix, x, w, 50, 10, big)
    alone, st0 = _run(ix, x, w, 50, 10, 0)
    _same(shared, alone)
    assert st["codes_scanned"] == st0["codes_scanned"] == 900 * w * 40 and st["codes_streamed"] < st0["codes_streamed"]


@pytest.mark.parametrize("c,w,m,ds", [(1025, 70, 8, 8), (8193, 70, 8, 16), (8193, 66, 16, 8)])
def test_kept_pairs_of_many_lists(c, w, m, ds):
    """The bound lists and counts the pairs that it keeps: more lists than one step of the grouping takes, more lists a query than one step
    of the plan, and more kept pairs than one round of the table kernel."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(c + m)
    d, n, nq, kp = m * ds, 2300, 2003, 60
    groups = c // 9     # of nine lists or more, near one another
    coarse = (rng.uniform(0, 100, (groups, d))[np.arange(c) % groups] + rng.normal(0, 4, (c, d))).astype(np.float32)
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, rng.normal(0, 12, (m, 256, ds)).astype(np.float32), None)
    ix.import_(np.arange(c + 1, dtype=np.int64) * n, rng.permutation(c * n).astype(np.int32), rng.integers(0, 256, (c * n, m), dtype=np.uint8))
    x = (coarse[rng.integers(0, c, nq)] + rng.normal(0, 12, (nq, d))).astype(np.float32)
    left, st = _run(ix, x, w, kp, 10, -1)
    alone, _ = _run(ix, x, w, kp, 10, 0)
    _same(left, alone)
    assert st["codes_scanned"] == nq * w * n >= 3e8 and st["dense_fallbacks"] == st["bound_retries"] == 0
    # 32 pairs to each of the table kernel's workgroups, at most 7 for 4 compute units
    kept = sum(st[p] for p in ("codes_scanned_shared", "codes_scanned_shared2", "codes_scanned_shared8")) / n
    assert 7168 < kept < 0.5 * nq * w, kept


@pytest.mark.parametrize("m,ds,kp", [(4, 32, 3000), (8, 16, 3000), (8, 32, 900), (16, 8, 3000)])
def test_samples_of_ragged_and_empty_lists(m, ds, kp):
    """Sets of pairs whose samples are empty, a single entry, a piece of 128 and one more, or hundreds of pieces; the last set is not full."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(m + ds)
    lens = np.array([0, 1, 127, 129, 4097, 90000, 60000, 30000, 20001, 0, 255, 70000, 3])
    c, d, n = len(lens), m * ds, int(lens.sum())
    coarse = rng.uniform(0, 60, (c, d)).astype(np.float32)
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, rng.normal(0, 12, (m, 256, ds)).astype(np.float32), None)
    ix.import_(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), rng.permutation(n).astype(np.int32),
               rng.integers(0, 256, (n, m)).astype(np.uint8))
    x = rng.uniform(0, 60, (1501, d)).astype(np.float32)
    left, st = _run(ix, x, c, kp, 20, -1)
    alone, _ = _run(ix, x, c, kp, 20, 0)
    _same(left, alone)
    assert st["dense_fallbacks"] == st["bound_retries"] == 0


def test_a_query_done_again_looks_at_every_list():
    """The lists begin with entries that are not like the rest: the bound from the sample lets through far more than fits, and
    the queries are scanned again pair by pair."""
    rng = np.random.default_rng(5)
    m, ds, c, n, w = 8, 16, 10, 50000, 6
    codes = rng.integers(0, 256, (c * n, m)).astype(np.uint8)
    near = rng.integers(0, 4, (c * n, m)).astype(np.uint8)
    late = (np.arange(c * n) % n) > n // 4
    codes[late] = near[late]
    ix, coarse, pq = _index(rng, m * ds, c, m, n, codes)
    x = (coarse[rng.integers(0, c, 1001)] + pq[:, 1].reshape(-1) + rng.normal(0, 3, (1001, m * ds))).astype(np.float32)
    ix.set_tuning(full_mult=1, cap_mult=1, min_cap=1)
    left, st = _run(ix, x, w, 50, 10, -1)
    alone, _ = _run(ix, x, w, 50, 10, 0)
    assert st["bound_retries"] > 0
    _same(left, alone)


def _small_inputs(rng, kind, c, nq):
    """d = 64, m = 8: "block": a sub-vector that is zero in every centroid and reproduction value, queries that hold next to nothing
    there.  "scaled": whole numbers times 2^-62, whose squares and sums are exact, while powers of two that bring residuals and
    reproduction values to what half precision holds are beyond fp32 together."""
    d, m = 64, 8
    if kind == "block":
        coarse = (50 + 6 * rng.normal(size=(c, d))).astype(np.float32)
        pq = rng.normal(0, 12, (m, 256, d // m)).astype(np.float32)
        x = (coarse[rng.integers(0, c, nq)] + rng.normal(0, 12, (nq, d))).astype(np.float32)
        coarse[:, -8:] = 0
        pq[-1] = 0
        x[:, -8:] = 0
        x[::20, -8] = 1e-37
        x[7::20, -3] = 1e-43
    else:
        unit = np.float32(2.0 ** -62)
        coarse = rng.integers(-5, 6, (c, d)) * unit
        pq = rng.integers(-8, 9, (m, 256, d // m)) * unit
        x = coarse[rng.integers(0, c, nq)] + np.round(rng.integers(-10, 11, (nq, d)) * rng.uniform(0, 1, (nq, 1))) * unit
    return coarse.astype(np.float32), pq.astype(np.float32), x.astype(np.float32)


@pytest.mark.parametrize("kind", ["block", "scaled"])
@pytest.mark.parametrize("lists", ["shared", "by query"])
def test_very_small_components(kind, lists):
    """Components near the end of fp32's range: no list is lost, of those queries or of the ones whose pairs are bounded beside them."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(17)
    c, w, kp = 12, 7, 60
    n, nq = (25001, 2000) if lists == "shared" else (2500, 300)
    coarse, pq, x = _small_inputs(rng, kind, c, nq)
    ix = pkg.Index(64, c, 8, 0)
    ix.set_codebooks(coarse, pq)
    ix.import_(np.arange(c + 1, dtype=np.int64) * n, rng.permutation(c * n).astype(np.int32), rng.integers(0, 256, (c * n, 8)).astype(np.uint8))
    ix.set_profiling(2)
    left, st = _run(ix, x, w, kp, 10, -1)
    t = ix.stage_times()
    assert (t["sample"] == 0) == (lists == "by query") and (t["scan_shared8"] > 0) == (lists == "shared")
    alone, _ = _run(ix, x, w, kp, 10, 0)
    _same(left, alone)
    assert st["dense_fallbacks"] == st["bound_retries"] == 0


@pytest.mark.parametrize("m,ds", [(4, 16), (8, 8), (16, 8)])
@pytest.mark.parametrize("table_mode", [0, 1])
def test_tables_below_what_half_precision_scales(m, ds, table_mode):
    """Whole numbers times 2^-66, entries of zero among them: 60000 over the largest sum of entries is beyond fp32, as are the powers of
    two for the operands of the units of 64; all units still keep what the scan of single pairs keeps."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(m)
    c, w, n, nq, d = 12, 7, 8001, 600, m * ds
    unit = np.float32(2.0 ** -66)
    coarse = rng.integers(-5, 6, (c, d)) * unit
    pq = rng.integers(-8, 9, (m, 256, ds)) * unit
    pq[:, 0] = 0
    x = coarse[rng.integers(0, c, nq)] + np.round(rng.integers(-10, 11, (nq, d)) * rng.uniform(0, 1, (nq, 1)) ** 3) * unit
    coarse, pq, x = (v.astype(np.float32) for v in (coarse, pq, x))
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, pq)
    ix.import_(np.arange(c + 1, dtype=np.int64) * n, rng.permutation(c * n).astype(np.int32), rng.integers(0, 256, (c * n, m)).astype(np.uint8))
    ix.set_table_mode(table_mode)
    alone, _ = _run(ix, x, w, 60, 10, 0)
    for mode in (1, 2, 3):
        shared, st = _run(ix, x, w, 60, 10, mode)
        assert st["codes_scanned_shared8"] + st["codes_scanned_shared64"] > 0 or mode == 1
        _same(shared, alone)


@pytest.mark.parametrize("lists", ["shared", "by query"])
def test_bounds_pause_where_little_is_left_out(lists):
    """Nine queries in ten lie where lists overlap: a call leaves out less than a seventh, the next fifteen of the same w and k' scan
    everything, the one after that tries again; other sizes and queries of which much is left out are not held up.  The results are the
    same throughout."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(23)
    d, m, c, w, kp = 64, 8, 36, 12, 60
    n, nq = (7001, 4000) if lists == "shared" else (1500, 400)
    coarse = rng.uniform(0, 100, (c, d)).astype(np.float32)
    coarse[:18] = coarse[0] + rng.normal(0, 0.5, (18, d))
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, rng.normal(0, 15, (m, 256, d // m)).astype(np.float32), None)
    ix.import_(np.arange(c + 1, dtype=np.int64) * n, rng.permutation(c * n).astype(np.int32), rng.integers(0, 256, (c * n, m)).astype(np.uint8))
    from_list = np.where(np.arange(nq) % 10 == 3, rng.integers(18, c, nq), 0)
    x = (coarse[from_list] + rng.normal(0, 15, (nq, d))).astype(np.float32)
    apart = (coarse[rng.integers(18, c, nq)] + rng.normal(0, 15, (nq, d))).astype(np.float32)

    def done(st):   # share of the estimates that were computed
        parts = ("codes_scanned_shared", "codes_scanned_shared2", "codes_scanned_shared8") if lists == "shared" else ("codes_streamed",)
        return sum(st[p] for p in parts) / st["codes_scanned"]

    alone, _ = _run(ix, x, w, kp, 10, 0)
    for call in range(18):
        left, st = _run(ix, x, w, kp, 10, -1)
        _same(left, alone)
        assert (6 / 7 < done(st) < 0.97) if call in (0, 16) else done(st) > 0.99, call
    assert done(_run(ix, x, w, kp + 1, 10, -1)[1]) < 0.97      # another k', in the middle of a pause
    alone, _ = _run(ix, apart, w, kp, 10, 0)
    for call in range(3):
        left, st = _run(ix, apart, w, kp, 10, -1)
        _same(left, alone)
        assert done(st) < 0.6
