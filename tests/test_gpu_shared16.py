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


@pytest.mark.parametrize("table_mode", [0, 1])
@pytest.mark.parametrize("m", [4, 8, 16])
def test_units_of_sixteen_give_the_same_bits(m, table_mode):
    rng = np.random.default_rng(100 + m)
    # ends of the 512-entry blocks and of the kernel's passes; every query visits every list
    lengths = [60000, 511, 512, 513, 1, 0, 30001]
    ix, _ = _index(rng, 64, len(lengths), m, lengths)
    ix.set_table_mode(table_mode)
    for nq in (8, 9, 15, 16, 17, 24, 25, 33):   # units: one of eight; one of sixteen with empty slots, full; and a rest beside it
        x = rng.uniform(0, 100, (nq, 64)).astype(np.float32)
        st = _check(ix, x, len(lengths), 20, 10)
        full = nq if nq % 16 == 0 or nq % 16 >= 5 else nq - nq % 16
        assert st["codes_scanned_shared8"] == full * sum(lengths), nq


@pytest.mark.parametrize("shape", ["far lists", "one value", "huge", "zeros"])
def test_units_of_sixteen_with_awkward_tables(shape):
    """Tables whose entries the 5-bit steps cannot tell apart, or that overflow: the filter must only ever let too much pass."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(3)
    d, c, m, n = 64, 3, 8, 40000
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
    x = rng.uniform(0, 100, (19, d)).astype(np.float32)
    if shape == "zeros":            # one entry in a hundred lies exactly at every query: bound and smallest estimate are 0
        coarse[:] = 0
        pq[:, 0] = 0
        codes[rng.permutation(c * n)[:c * n // 100]] = 0
        x[:] = 0
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, pq)
    ix.import_(np.arange(c + 1) * n, rng.permutation(c * n).astype(np.int32), codes)
    st = _check(ix, x, c, 25, 25)
    assert st["codes_scanned_shared8"] > 0
