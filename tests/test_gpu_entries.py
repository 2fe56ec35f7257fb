"""Import and export of the inverted file: the dense arrays come back as they went in, whatever the lists look like."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c,N,m,mr,occupied", [
    (1, 1, 8, 0, 1.0),              # one entry
    (7, 0, 8, 8, 1.0),              # none
    (5000, 300, 4, 4, 0.01),        # a workgroup's entries far apart, thousands of empty lists between them
    (64, 4097, 16, 16, 0.5),
    (1000, 70001, 64, 32, 1.0),
    (300, 1_200_000, 64, 8, 0.9),   # more code bytes than one copy takes
])
def test_import_export_round_trip(c, N, m, mr, occupied):
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(c + N)
    d = {4: 32, 8: 64, 16: 64, 32: 64, 64: 64}[m]
    lists = np.sort(rng.choice(np.flatnonzero(rng.random(c) < occupied) if occupied < 1 else np.arange(c), N)) if N else np.empty(0, int)
    offsets = np.zeros(c + 1, dtype=np.int64)
    np.cumsum(np.bincount(lists, minlength=c), out=offsets[1:])
    ids = rng.permutation(N).astype(np.int32)
    codes = rng.integers(0, 256, (N, m)).astype(np.uint8)
    rcodes = rng.integers(0, 256, (N, mr)).astype(np.uint8)
    ix = pkg.Index(d, c, m, mr)
    ix.set_codebooks(rng.random((c, d)), rng.random((m, 256, d // m)), rng.random((mr, 256, d // mr)) if mr else None)
    ix.import_(offsets, ids, codes, rcodes if mr else None)
    for got, want in zip(ix.export(), (offsets, ids, codes, rcodes)):
        assert got.shape == want.shape and (got == want).all()


def test_export_where_room_is_short():
    """A memory limit that leaves room for a small buffer only: more copies, the same arrays."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(3)
    N, c = 400_000, 50
    offsets = np.linspace(0, N, c + 1).astype(np.int64)
    ids, codes = rng.permutation(N).astype(np.int32), rng.integers(0, 256, (N, 8)).astype(np.uint8)
    ix = pkg.Index(64, c, 8, 0)
    ix.set_codebooks(rng.random((c, 64)), rng.random((8, 256, 8)))
    ix.import_(offsets, ids, codes)
    held = sum(ix.workspace_info()[k] for k in ("index_bytes", "workspace_bytes", "pool_bytes"))
    ix.set_memory_limit(held + 200_000)
    got = ix.export()
    assert (got[0] == offsets).all() and (got[1] == ids).all() and (got[2] == codes).all()
    ix.set_memory_limit(held + 1000)
    with pytest.raises(pkg.IvfrError) as e:
        ix.export()
    assert e.value.code == pkg.binding.ERR_OOM


def test_small_index_where_room_is_short():
    """2000 entries with wide codes under a limit that leaves 20 KB: less than one array's 128 KB, and than half of it."""
    import paper_1102_3828_amd as pkg
    rng = np.random.default_rng(4)
    N, c = 2000, 3
    offsets = np.array([0, 700, 700, N])
    ids, codes = rng.permutation(N).astype(np.int32), rng.integers(0, 256, (N, 64)).astype(np.uint8)
    books = rng.random((c, 64)), rng.random((64, 256, 1))
    ix = pkg.Index(64, c, 64, 0)
    ix.set_codebooks(*books)
    ix.import_(offsets, ids, codes)
    held = ix.workspace_info()["index_bytes"]
    ix.set_memory_limit(held + 20_000)
    for got, want in zip(ix.export(), (offsets, ids, codes)):
        assert (got == want).all()
    again = pkg.Index(64, c, 64, 0)
    again.set_codebooks(*books)
    again.set_memory_limit(held + 20_000)
    again.import_(offsets, ids, codes)
    for got, want in zip(again.export(), (offsets, ids, codes)):
        assert (got == want).all()
