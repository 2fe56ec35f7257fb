"""The selections at the sizes where they change from registers to sweeps over memory, with whole-number codebooks: estimates are
exact, many of them equal, and the short-list and the results are known to the last tie."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("distinct", [3, 200])
@pytest.mark.parametrize("n,kp,k", [
    (97, 96, 10), (513, 512, 96), (1025, 1000, 256), (2049, 2047, 300), (2100, 2048, 10), (2100, 2049, 97),   # final: 2048 keys
    (4095, 2000, 100), (4096, 4095, 100), (4097, 4096, 129), (4097, 96, 96),                                 # short-list: 4096 records
    (13311, 10239, 10), (13312, 10240, 300), (13313, 10241, 128),                                             # 13312; final: 10240
])
def test_short_list_and_results_to_the_last_tie(n, kp, k, distinct):
    import torch
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(n + kp)
    d, m = 32, 4
    coarse = np.zeros((1, d), np.float32)
    pq = rng.integers(-20, 21, (m, 256, d // m)).astype(np.float32)
    codes = rng.integers(0, distinct, (n, m)).astype(np.uint8)
    ids = rng.permutation(n).astype(np.int32)
    x = rng.integers(-30, 31, (5, d)).astype(np.float32)
    ix = pkg.Index(d, 1, m, 0)
    ix.set_codebooks(coarse, pq, None)
    ix.import_(np.array([0, n], np.int64), ids, codes)
    y = np.concatenate([pq[j][codes[:, j]] for j in range(m)], 1).astype(np.float64)
    est = ((x[:, None, :].astype(np.float64) - y[None]) ** 2).sum(-1)
    for mode, full in ((0, 1000), (-1, 8), (0, 1)):   # everything kept; as the call chooses; a bound where that pays
        ix.set_list_sharing(mode)
        ix.set_tuning(full_mult=full)
        g_ids, g_dist, t = ix.search(torch.from_numpy(x).cuda(), 1, kp, k, trace=True)
        s_ids = t["short_ids"].cpu().numpy()
        for q in range(len(x)):
            order = np.lexsort((ids, est[q]))
            assert set(s_ids[q].tolist()) == set(ids[order[:kp]].tolist())
            assert (g_ids[q].cpu().numpy() == ids[order[:k]]).all()
            assert (g_dist[q].cpu().numpy() == est[q][order[:k]]).all()
    ix.close()


@pytest.mark.parametrize("c", [2047, 2048, 2049, 8191, 8192, 8193])
@pytest.mark.parametrize("w", [1, 257, 300])
def test_visited_lists_to_the_last_tie(c, w):
    """The probe at the sizes where its kernel changes: up to 2048 and up to 8192 lists in registers, more from memory."""
    import torch
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(c + w)
    d, m = 32, 4
    coarse = rng.integers(0, 3, (c, d)).astype(np.float32)
    coarse[:, 8:] = 0                                  # 3^8 centroids at the most: many are there more than once
    x = rng.integers(-2, 5, (5, d)).astype(np.float32)
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse, rng.normal(0, 1, (m, 256, d // m)).astype(np.float32), None)
    ix.import_(np.arange(c + 1, dtype=np.int64), np.arange(c, dtype=np.int32), rng.integers(0, 256, (c, m)).astype(np.uint8))
    _, _, t = ix.search(torch.from_numpy(x).cuda(), w, 10, 1, trace=True)
    dist = ((x[:, None, :].astype(np.int64) - coarse[None].astype(np.int64)) ** 2).sum(-1)
    want = np.argsort(dist, axis=1, kind="stable")[:, :w]
    assert (t["probe"].cpu().numpy() == want).all()
    assert (t["probe_dist"].cpu().numpy() == np.take_along_axis(dist, want, 1)).all()
    ix.close()


@pytest.mark.parametrize("n,kp,k", [(15400, 10300, 50), (19000, 12000, 20)])   # from memory: twelve, four and one load at a time
def test_short_list_from_memory_to_the_last_tie(n, kp, k):
    test_short_list_and_results_to_the_last_tie(n, kp, k, 200)


@pytest.mark.parametrize("d,c,w", [(32, 1, 1), (32, 3, 2), (64, 255, 255), (64, 256, 256), (64, 257, 256), (128, 257, 8), (128, 512, 1),
                                   (128, 513, 64), (256, 1000, 13), (256, 1024, 100), (512, 1023, 7), (512, 1024, 255), (128, 1025, 8)])
def test_visited_lists_of_a_few_queries_are_those_of_many(d, c, w):
    """Up to a query per compute unit and up to 1024 centroids of 32 to 512 dimensions distances and selection are one kernel: the same
    lists and the same bits as in a batch that goes through the matrix cores; the neighbours of the limit take that way anyway."""
    import torch
    import paper_1102_3828_amd as pkg
    g = torch.Generator(device="cuda").manual_seed(d + c + w)
    m = max(4, d // 32)
    coarse = 30.0 * torch.randn((c, d), generator=g, device="cuda")
    x = coarse[torch.randint(c, (600,), generator=g, device="cuda")] + 10.0 * torch.randn((600, d), generator=g, device="cuda")
    ix = pkg.Index(d, c, m, 0)
    ix.set_codebooks(coarse.cpu().numpy(), torch.randn((m, 256, d // m), generator=g, device="cuda").cpu().numpy(), None)
    ix.import_(np.arange(c + 1, dtype=np.int64), np.arange(c, dtype=np.int32), np.zeros((c, m), np.uint8))
    many = ix.search(x, w, 10, 1, trace=True)[2]
    for a, b in ((0, 1), (1, 38), (38, 200), (200, 456), (456, 600)):
        few = ix.search(x[a:b].contiguous(), w, 10, 1, trace=True)[2]
        assert torch.equal(few["probe"], many["probe"][a:b])
        assert torch.equal(few["probe_dist"].view(torch.int32), many["probe_dist"][a:b].view(torch.int32))
    with pytest.raises(pkg.IvfrError):
        y = x[:7].clone()
        y[5, d - 1] = float("nan")
        ix.search(y, w, 10, 1)
    ix.close()
