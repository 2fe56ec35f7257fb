"""What a program that uses this library has it do, as a list of measurable cases.

Three kinds of pass, each through the public entry points of the package:
  search   Index.search (or Index.search_static) on a finished index: the query stage, from one
           interactive query to batches of a thousand, per-list lengths from hundreds to 10^5 entries
  build    create an index, set its codebooks, add uint8 vectors, finalize, export the inverted file
           (what a program does that builds an index and saves it)
  train    learn the three quantizers on uint8 vectors and read the codebooks back

A search case's index is imported: lists, ids and codes are drawn directly with the statistics that an
encoded clustered database has (neighbouring lists that share a cluster, code bytes distributed like the
codes of Gaussian residuals, list lengths scattered as trained lists are), so that no vectors have to be
encoded to prepare it.  Everything is drawn from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1102_3828_amd as pkg

DEV = "cuda:0"
KS = 256              # reproduction values per sub-quantizer
CENTROID_SPREAD = 10.0   # of the centroids of one cluster around its centre, per dimension
RESIDUAL_SIGMA = 17.0    # of an entry around its list's centroid, per dimension


def _search(name, N, c, w, kp, k, nq, m=8, mr=8, d=128, skew=0.7, table=0, static=False):
    return {"name": name, "kind": "search", "N": N, "c": c, "w": w, "kp": kp, "k": k, "nq": nq, "m": m, "mr": mr, "d": d,
            "skew": skew, "table": table, "static": static}


def listed():
    return [
        # one interactive query against a small index: launches and latency
        _search("one_query", 100_000, 256, 8, 100, 10, 1, skew=0.0),
        # the smallest workload of the benchmark: 100 queries, 10^5 vectors
        _search("small_batch", 100_000, 256, 8, 100, 10, 100, skew=0.0),
        # a serving loop that must not allocate: a few dozen queries through the fixed-workspace entry point
        _search("static_serving", 1_000_000, 1024, 8, 500, 50, 37, static=True),
        # 10^6 vectors, 1000 queries, 16 refinement bytes (second workload of the benchmark)
        _search("batch_1e6", 1_000_000, 1024, 8, 1000, 100, 1000, mr=16, skew=0.0),
        # 10^7 vectors in 8192 lists, 32 refinement bytes (third workload of the benchmark)
        _search("batch_1e7", 10_000_000, 8192, 16, 1000, 100, 1000, mr=32, skew=0.0),
        # long short-lists on medium lists: k' = 10000 of 64 lists (fourth workload, at a third of its vectors)
        _search("long_shortlist", 30_000_000, 8192, 64, 10_000, 100, 1000, mr=16),
        # long lists (10^5 entries) shared by many queries: the large workload's scan at a tenth of its vectors
        _search("long_lists", 100_000_000, 1024, 64, 1000, 100, 1000),
        # odd sizes everywhere: plain IVFADC, 64 dimensions, 16 code bytes, split look-up tables
        _search("odd_split_tables", 777_777, 1000, 13, 333, 37, 501, m=16, mr=0, d=64, table=1),
        # thousands of results per query (the paper's own k' / k = 2) with wide codes
        _search("many_results", 3_000_000, 1024, 32, 10_000, 5000, 100, m=32, mr=32),
        # building and saving an index: 10^6 vectors, 1024 lists; 3*10^6 vectors, 8192 lists
        {"name": "build_1e6", "kind": "build", "N": 1_000_000, "c": 1024, "m": 8, "mr": 16, "d": 128},
        {"name": "build_many_lists", "kind": "build", "N": 3_000_001, "c": 8192, "m": 8, "mr": 8, "d": 128},
        # learning the quantizers of the 10^6-vector index on 10^5 vectors (few Lloyd iterations: a vector between two
        # centroids that rounding sends the other way moves both, and that grows from iteration to iteration)
        {"name": "train_1e5", "kind": "train", "n": 100_000, "c": 1024, "m": 8, "mr": 16, "d": 128, "iters": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a search four times out of six, else a build or a training."""
    kind = rng.choice(["search", "search", "search", "search", "build", "train"])
    d = rng.choice([64, 128, 128, 128, 256])
    m = rng.choice([v for v in (4, 8, 8, 8, 16, 32, 64) if d // 32 <= v <= d])
    mr = rng.choice([v for v in (0, 8, 8, 16, 16, 32) if v == 0 or d // 32 <= v])
    if kind == "build":
        return {"kind": "build", "N": _log_int(rng, 20_000, 2_000_000), "c": _log_int(rng, 64, 4096), "m": m, "mr": mr, "d": d}
    if kind == "train":
        # one iteration: a vector sent the other way in a first one is not followed by others
        c = _log_int(rng, 64, 1024)
        m = {64: 4, 128: 8, 256: 16}[d] * rng.choice([1, 1, 2])
        return {"kind": "train", "n": _log_int(rng, 30_000, 100_000), "c": c, "m": m, "mr": 0, "d": d, "iters": 1}
    c = _log_int(rng, 64, 8192)
    N = _log_int(rng, 100 * c, max(200 * c, min(20_000_000, 20_000 * c)))
    w = _log_int(rng, 1, min(64, c))
    visited = max(1, w * N // c)
    kp = _log_int(rng, 20, max(40, min(10_000, visited // 3)))
    k = _log_int(rng, 1, min(kp, 2000))
    nq = _log_int(rng, 1, max(2, min(1500, 2_000_000_000 // visited, 4_000_000 // kp)))
    static = rng.random() < 0.25 and nq * kp < 200_000 and nq * w * m < 50_000
    table = 1 if rng.random() < 0.25 and not static else 0
    return {"kind": "search", "N": N, "c": c, "w": w, "kp": kp, "k": k, "nq": nq, "m": m, "mr": mr, "d": d,
            "skew": rng.choice([0.0, 0.7]), "table": table, "static": static}


# ---- inputs -----------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _nearest_codeword(v, book):
    """Index of the nearest row of book [256, ds] for each row of v [n, ds] (elementwise, so the same every time)."""
    return torch.cat([((b[:, None, :] - book[None, :, :]) ** 2).sum(-1).argmin(1) for b in v.split(4096)])


def _search_inputs(case, seed):
    """Codebooks, inverted file and queries of a search case, on the GPU."""
    g = _gen(seed)
    d, c, m, mr, N, nq = case["d"], case["c"], case["m"], case["mr"], case["N"], case["nq"]
    n_clusters = max(1, c // 4)
    centres = torch.rand((n_clusters, d), generator=g, device=DEV) * 100.0
    coarse = centres[torch.arange(c, device=DEV) % n_clusters] + CENTROID_SPREAD * torch.randn((c, d), generator=g, device=DEV)
    ds, dr = d // m, (d // mr if mr else 0)
    pq = 0.8 * RESIDUAL_SIGMA * torch.randn((m, KS, ds), generator=g, device=DEV)
    # codes of a pool of Gaussian residuals; an entry takes each block of dimensions from a row of the pool
    pool_n = 8192
    pool = RESIDUAL_SIGMA * torch.randn((pool_n, d), generator=g, device=DEV)
    code_pool = torch.empty((pool_n, m), dtype=torch.uint8, device=DEV)
    for j in range(m):
        v = pool[:, j * ds:(j + 1) * ds]
        code = _nearest_codeword(v, pq[j])
        code_pool[:, j] = code.to(torch.uint8)
        pool[:, j * ds:(j + 1) * ds] = v - pq[j][code]
    rq = None
    rcode_pool = None
    if mr:
        rq = 0.8 * pool.std() * torch.randn((mr, KS, dr), generator=g, device=DEV)
        rcode_pool = torch.empty((pool_n, mr), dtype=torch.uint8, device=DEV)
        for j in range(mr):
            rcode_pool[:, j] = _nearest_codeword(pool[:, j * dr:(j + 1) * dr], rq[j]).to(torch.uint8)
    blocks = d // max(ds, dr)
    code_pool = code_pool.reshape(pool_n, blocks, m // blocks)
    if mr:
        rcode_pool = rcode_pool.reshape(pool_n, blocks, mr // blocks)
    codes = torch.empty((N, m), dtype=torch.uint8, device=DEV)
    rcodes = torch.empty((N, mr), dtype=torch.uint8, device=DEV)
    b_idx = torch.arange(blocks, device=DEV)[None, :]
    step = max(1, (1 << 26) // blocks)
    for a in range(0, N, step):
        n = min(step, N - a)
        row = torch.randint(pool_n, (n, blocks), generator=g, device=DEV)
        codes[a:a + n] = code_pool[row, b_idx].reshape(n, m)
        if mr:
            rcodes[a:a + n] = rcode_pool[row, b_idx].reshape(n, mr)
        del row
    # list lengths, and ids ascending inside every list
    weights = torch.exp(case["skew"] * torch.randn((c,), generator=g, device=DEV)).double()
    counts = torch.floor(N * weights / weights.sum()).long()
    counts[0] += N - counts.sum()
    offsets = torch.zeros(c + 1, dtype=torch.int64, device=DEV)
    offsets[1:] = torch.cumsum(counts, 0)
    labels = torch.repeat_interleave(torch.arange(c, device=DEV, dtype=torch.int32), counts)
    labels = labels[torch.randperm(N, generator=g, device=DEV)]
    ids = torch.sort(labels, stable=True)[1].to(torch.int32)
    del labels
    # queries come from the database's clusters, a cluster as often as its lists are long; byte-valued components
    q_list = torch.searchsorted(offsets[1:], torch.randint(N, (nq,), generator=g, device=DEV), right=True)
    queries = coarse[q_list] + RESIDUAL_SIGMA * torch.randn((nq, d), generator=g, device=DEV)
    queries = queries.round().clamp(0.0, 255.0).contiguous()
    return {"coarse": coarse, "pq": pq, "rq": rq, "offsets": offsets, "ids": ids, "codes": codes, "rcodes": rcodes, "queries": queries}


def _byte_vectors(g, n, d, n_clusters):
    """uint8 [n, d] from a Gaussian mixture; returns the vectors and the mixture's centres."""
    centres = torch.rand((n_clusters, d), generator=g, device=DEV) * 100.0
    out = torch.empty((n, d), dtype=torch.uint8, device=DEV)
    for a in range(0, n, 1 << 20):
        b = min(n, a + (1 << 20))
        comp = torch.randint(n_clusters, (b - a,), generator=g, device=DEV)
        v = centres[comp] + 20.0 * torch.randn((b - a, d), generator=g, device=DEV)
        out[a:b] = v.round().clamp(0.0, 255.0).to(torch.uint8)
    return out, centres


def _build_inputs(case, seed):
    """Vectors and byte-valued codebooks.  With whole numbers in vectors and codebooks every distance is a whole number
    below 2^24, so nearest centroids and codes are the same in any correct arithmetic (ties go to the lowest index)."""
    g = _gen(seed)
    d, c, m, mr = case["d"], case["c"], case["m"], case["mr"]
    x, centres = _byte_vectors(g, case["N"], d, max(1, c // 2))
    coarse = (centres[torch.arange(c, device=DEV) % len(centres)] + CENTROID_SPREAD * torch.randn((c, d), generator=g, device=DEV))
    coarse = coarse.round().clamp(0.0, 255.0)
    pq = (16.0 * torch.randn((m, KS, d // m), generator=g, device=DEV)).round().clamp(-128.0, 127.0)
    rq = (9.0 * torch.randn((mr, KS, d // mr), generator=g, device=DEV)).round().clamp(-128.0, 127.0) if mr else None
    return {"x": x, "coarse": coarse, "pq": pq, "rq": rq}


def _np(t):
    return None if t is None else t.cpu().numpy()


def prepare(case, seed):
    if case["kind"] == "train":
        x, _ = _byte_vectors(_gen(seed), case["n"], case["d"], max(1, case["n"] // 100))
        return {"case": case, "x": x, "ix": pkg.Index(case["d"], case["c"], case["m"], case["mr"])}
    if case["kind"] == "build":
        s = _build_inputs(case, seed)
        return {"case": case, "x": s["x"], "books": (_np(s["coarse"]), _np(s["pq"]), _np(s["rq"]))}
    s = _search_inputs(case, seed)
    ix = pkg.Index(case["d"], case["c"], case["m"], case["mr"])
    ix.set_codebooks(_np(s["coarse"]), _np(s["pq"]), _np(s["rq"]))
    ix.import_(_np(s["offsets"]), _np(s["ids"]), _np(s["codes"]), _np(s["rcodes"]) if case["mr"] else None)
    ix.set_table_mode(case["table"])
    state = {"case": case, "ix": ix, "queries": s["queries"]}
    if case["static"]:
        state["ids"] = torch.empty((case["nq"], case["k"]), dtype=torch.int32, device=DEV)
        state["dist"] = torch.empty((case["nq"], case["k"]), dtype=torch.float32, device=DEV)
    del s
    torch.cuda.empty_cache()
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "train":
        state["ix"].train(state["x"], iters=case["iters"], seed=1)
        return [b for b in state["ix"].get_codebooks() if b is not None]
    if case["kind"] == "build":
        ix = pkg.Index(case["d"], case["c"], case["m"], case["mr"])
        ix.set_codebooks(*state["books"])
        ix.add(state["x"], 0)
        ix.finalize()
        out = ix.export()
        ix.close()
        return [a for a in out if a.size]
    if case["static"]:
        state["ix"].search_static(state["queries"], case["w"], case["kp"], case["k"], state["ids"], state["dist"])
        return state["ids"], state["dist"]
    return state["ix"].search(state["queries"], case["w"], case["kp"], case["k"])


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def work(case):
    c, d, m, mr = case["c"], case["d"], case["m"], case["mr"]
    books = 4 * (c * d + KS * d + (KS * d if mr else 0))
    if case["kind"] == "train":
        # every iteration looks at every vector: distances to the c centroids, then to the 256 values of each sub-quantizer
        n, it = case["n"], case["iters"]
        return {"bytes": n * d + books, "flops": n * it * 2 * d * (c + KS + (KS if mr else 0))}
    if case["kind"] == "build":
        N = case["N"]
        return {"bytes": N * d + books + N * (m + mr + 4) + 8 * (c + 1), "flops": N * 2 * d * (c + KS + (KS if mr else 0))}
    nq, w, N, kp, k = case["nq"], case["w"], case["N"], case["kp"], case["k"]
    visited = nq * w * N / c                                    # estimates of a pass
    distinct = N * (1.0 - math.exp(-nq * w / c))                # entries of lists that some query visits
    short = nq * min(kp, w * N / c)
    bytes_ = 4 * nq * d + books + distinct * m + short * (m + mr + 8) + 8 * nq * k
    flops = 2 * nq * c * d + 2 * nq * w * KS * d + visited * m + short * 4 * d
    return {"bytes": int(bytes_), "flops": int(flops)}


def tolerance(case):
    if case["kind"] == "build":
        return "exact"
    if case["kind"] == "train":
        # a vector halfway between two centroids may go either way: one such changes a codebook by up to 1e-3 and the
        # refinement codebook learned after it by 5e-3 (seen against 64 bits; without one, 2e-8)
        return {"rel": 2e-2}
    # distances agree to 5e-8; an entry at the edge of the short-list may be in or out of it and then shifts the
    # query's later ranks by one (3.5e-5 over a thousand queries)
    return {"rel": 2e-4, "differ": 5e-3}


# ---- the same results in 64 bits --------------------------------------------------------------------------------

def _mix64(z):
    with np.errstate(over="ignore"):
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _start_rows(seed, salt, n, count):
    """Training rows that a k-means starts from: those with the `count` smallest hashes of (seed, salt, row), in order."""
    golden = np.uint64(0x9E3779B97F4A7C15)
    with np.errstate(over="ignore"):
        key = _mix64(np.uint64(seed) * golden + np.uint64(salt))
        h = _mix64(key + np.arange(1, n + 1, dtype=np.uint64) * golden)
    return torch.from_numpy(np.sort(np.argsort(h, kind="stable")[:count])).to(DEV)


def _nearest64(x, cent):
    """Nearest row of cent for each row of x (float64, lowest index among equals)."""
    cn = (cent * cent).sum(1)
    ct = cent.T.contiguous()
    return torch.cat([(cn[None, :] - 2.0 * (b @ ct)).argmin(1) for b in x.split(max(1, (1 << 27) // len(cent)))])


def _lloyd64(x, cent, iters):
    for _ in range(iters):
        a = _nearest64(x, cent)
        s = torch.zeros_like(cent).index_add_(0, a, x)
        n = torch.bincount(a, minlength=len(cent))
        cent = torch.where(n[:, None] > 0, s / n.clamp(min=1)[:, None], cent)
    return cent


def _product64(x, parts, iters, salt0):
    """Codebook of a product quantizer on the rows of x, and what it leaves of them."""
    n, d = x.shape
    ds = d // parts
    book, rest = [], x.clone()
    for j in range(parts):
        v = x[:, j * ds:(j + 1) * ds].contiguous()
        cent = _lloyd64(v, v[_start_rows(1, salt0 + j, n, KS)].clone(), iters).float().double()
        book.append(cent)
        rest[:, j * ds:(j + 1) * ds] = v - cent[_nearest64(v, cent)]
    return torch.stack(book), rest


def _encode64(x, book):
    """Codes of the rows of x, and what they leave of them."""
    codes, rest = [], x.clone()
    ds = book.shape[2]
    for j in range(len(book)):
        v = x[:, j * ds:(j + 1) * ds].contiguous()
        k = _nearest64(v, book[j])
        codes.append(k.to(torch.uint8))
        rest[:, j * ds:(j + 1) * ds] = v - book[j][k]
    return torch.stack(codes, 1), rest


def _exact_train(case, seed):
    x = _byte_vectors(_gen(seed), case["n"], case["d"], max(1, case["n"] // 100))[0].double()
    cent = _lloyd64(x, x[_start_rows(1, 1, case["n"], case["c"])].clone(), case["iters"]).float().double()
    x = x - cent[_nearest64(x, cent)]
    pq, rest = _product64(x, case["m"], case["iters"], 100)
    out = [cent, pq]
    if case["mr"]:
        out.append(_product64(rest, case["mr"], case["iters"], 200)[0])
    return [o.cpu().numpy() for o in out]


def _exact_build(case, seed):
    s = _build_inputs(case, seed)
    lists, codes, rcodes = [], [], []
    coarse, pq = s["coarse"].double(), s["pq"].double()
    for xb in s["x"].split(1 << 19):
        x = xb.double()
        a = _nearest64(x, coarse)
        lists.append(a)
        cb, rest = _encode64(x - coarse[a], pq)
        codes.append(cb)
        if case["mr"]:
            rcodes.append(_encode64(rest, s["rq"].double())[0])
    lists = torch.cat(lists)
    ids = torch.sort(lists, stable=True)[1]
    offsets = torch.zeros(case["c"] + 1, dtype=torch.int64, device=DEV)
    offsets[1:] = torch.cumsum(torch.bincount(lists, minlength=case["c"]), 0)
    out = [offsets, ids.to(torch.int32), torch.cat(codes)[ids]]
    if case["mr"]:
        out.append(torch.cat(rcodes)[ids])
    return [o.cpu().numpy() for o in out]


def _exact_search(case, seed):
    s = _search_inputs(case, seed)
    d, m, mr, w, kp, k = case["d"], case["m"], case["mr"], case["w"], case["kp"], case["k"]
    coarse, pq = s["coarse"].double(), s["pq"].double()
    rq = s["rq"].double() if mr else None
    starts, lengths = s["offsets"][:-1], s["offsets"][1:] - s["offsets"][:-1]
    jm, jr = torch.arange(m, device=DEV), torch.arange(max(mr, 1), device=DEV)
    ids_out = torch.full((case["nq"], k), -1, dtype=torch.int32, device=DEV)
    dist_out = torch.full((case["nq"], k), float("inf"), dtype=torch.float64, device=DEV)
    for q in range(case["nq"]):
        x = s["queries"][q].double()
        dc = ((x[None, :] - coarse) ** 2).sum(1)
        probe = torch.sort(dc, stable=True)[1][:w]
        tables = (((x[None, :] - coarse[probe]).reshape(w, m, 1, d // m) - pq[None]) ** 2).sum(-1)
        length = lengths[probe]
        rank = torch.repeat_interleave(torch.arange(w, device=DEV), length)     # of its list among the w, for each entry
        lst = probe[rank]
        pos = starts[lst] + torch.arange(len(lst), device=DEV) - (torch.cumsum(length, 0) - length)[rank]
        if len(pos) == 0:
            continue
        code = s["codes"][pos].int()
        est = tables[rank, 0, code[:, 0]]
        for j in range(1, m):
            est += tables[rank, j, code[:, j]]
        if len(est) > kp:
            keep = torch.topk(est, kp, largest=False)[1]
            pos, lst = pos[keep], lst[keep]
        y = coarse[lst] + pq[jm[None, :], s["codes"][pos].long()].reshape(len(pos), d)
        if mr:
            y = y + rq[jr[None, :], s["rcodes"][pos].long()].reshape(len(pos), d)
        ref = ((x[None, :] - y) ** 2).sum(1)
        ident = s["ids"][pos]
        order = torch.sort(ident)[1]
        ref, ident = ref[order], ident[order]
        order = torch.sort(ref, stable=True)[1][:k]
        ids_out[q, :len(order)] = ident[order]
        dist_out[q, :len(order)] = ref[order]
    return ids_out.cpu(), dist_out.cpu()


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "build":
        return _exact_build(case, seed)
    visited = case["w"] * case["N"] / case["c"]
    if case["nq"] * (3e-3 + visited * (5e-10 + 1e-10 * case["m"])) > 20.0:   # about its seconds on one GPU
        return None
    return _exact_search(case, seed)
