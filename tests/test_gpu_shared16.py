"""Units of sixteen queries on 5-bit tables against the per-pair scan: the recorded estimates are re-evaluated in fp32, so
short-lists and results are the same bits, whatever the tables look like and however full the last unit of a list is."""
import numpy as np
import pytest

from test_gpu_scan_select import _index

pytestmark = pytest.mark.gpu


def _check(ix, x, w, kp, k):
    import torch
    xq = torch.from_numpy(x).cuda()
    out = []
    for mode in (2, 0):
        ix.set_list_sharing(mode)
        ids, dist, t = ix.search(xq, w, kp, k, trace=True)
        n = t["short_count"].cpu().numpy()
        s_ids, s_est = t["short_ids"].cpu().numpy(), t["short_est"].cpu().numpy()
        short = [sorted(zip(s_est[q, :n[q]].tolist(), s_ids[q, :n[q]].tolist())) for q in range(len(x))]
        out.append((ids.cpu().numpy(), dist.cpu().numpy(), n, short, ix.search_stats()))
    a, b = out
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and (a[2] == b[2]).all() and a[3] == b[3]
    assert a[4]["dense_fallbacks"] == b[4]["dense_fallbacks"]   # no survivor was lost to the filter
    assert a[4]["codes_scanned"] == b[4]["codes_scanned"] and b[4]["codes_scanned_shared8"] == 0
    return a[4]


# what the units of sixteen ask for: lists of 4 10^4 entries on average (as visited), 2 10^9 estimates a batch, few that pass
QUERIES, KP = 11200, 16


@pytest.mark.parametrize("table_mode", [0, 1])
@pytest.mark.parametrize("rest", [0, 4, 5, 8, 9, 12, 15])
def test_units_of_sixteen_give_the_same_bits(rest, table_mode):
    rng = np.random.default_rng(100 + rest)
    # ends of the 512-entry blocks and of the kernel's passes; every query visits every list
    lengths = [60000, 511, 512, 513, 1, 0, 60001, 59999]
    ix, _ = _index(rng, 64, len(lengths), 8, lengths)
    ix.set_table_mode(table_mode)
    nq = QUERIES + rest
    x = rng.uniform(0, 100, (nq, 64)).astype(np.float32)
    st = _check(ix, x, len(lengths), KP, 10)
    # units of sixteen, the last one with empty slots from nine on; a rest of five to eight is a unit of eight.  (Units of eight
    # alone would leave one to four of the rests nine and twelve to other units.)
    assert st["codes_scanned_shared8"] == (nq if rest == 0 or rest >= 5 else nq - rest) * sum(lengths)


@pytest.mark.parametrize("m,nq,kp,n", [
    (4, QUERIES + 9, KP, 60000), (16, QUERIES + 9, KP, 60000),     # other code widths
    (8, 2000 + 9, KP, 60000),                                     # too little work
    (8, QUERIES + 9, 40, 60000),                                  # too many estimates pass
    (8, 16000 + 9, KP, 30000),                                    # short lists
])
def test_other_batches_stay_with_units_of_eight(m, nq, kp, n):
    rng = np.random.default_rng(m + nq)
    ix, _ = _index(rng, 64, 5, m, [n] * 5)
    st = _check(ix, rng.uniform(0, 100, (nq, 64)).astype(np.float32), 5, kp, 10)
    assert st["codes_scanned_shared8"] == (nq - nq % 8) * 5 * n


@pytest.mark.parametrize("shape", ["far lists", "one value", "huge", "zeros"])
def test_units_of_sixteen_with_awkward_tables(shape):
    """Tables whose entries the 5-bit steps cannot tell apart, or that overflow: the filter must only ever let too much pass."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(3)
    d, c, m, n = 64, 3, 8, 60000
    coarse = rng.uniform(0, 100, (c, d)).astype(np.float32)
    pq = rng.normal(0, 15, (m, 256, d // m)).astype(np.float32)
    if shape == "far lists":
        coarse[1] += 1.0e4          # every estimate of list 1 lies beyond every bound
        coarse[2] = coarse[0]       # and lists 0 and 2 tie but for their codes
    elif shape == "one value":
        pq[:4] = pq[:4, :1]         # half of the sub-quantizers contribute a constant
    elif shape == "huge":
        pq *= 1.0e16                # estimates of 1e34 and more
    codes = rng.integers(0, 256, (c * n, m)).astype(np.uint8)
    x = rng.uniform(0, 100, (QUERIES + 9, d)).astype(np.float32)
    if shape == "zeros":            # one entry in a hundred lies exactly at every query: bound and smallest estimate are 0
        coarse[:] = 0
        pq[:, 0] = 0
        codes[rng.permutation(c * n)[:c * n // 100]] = 0
        x[:] = 0
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, pq)
    ix.import_(np.arange(c + 1) * n, rng.permutation(c * n).astype(np.int32), codes)
    st = _check(ix, x, c, KP, KP)
    assert st["codes_scanned_shared8"] == len(x) * c * n     # the rest of nine included: units of sixteen
