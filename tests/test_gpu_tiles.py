"""Heavy rows accumulated from the chunk-major copy of B (the default path of
rows of more than 3456 products when a row's entries meet a chunk of 2^14
columns with one product or more on average; test_rule has the rule's lines), at
the sizes where it can go wrong: column counts around whole chunks and whole groups of 16 chunks, every
region size (one wave up to the dense accumulator), parts long enough to be
shared by a work group's waves (and more of them than the shared list holds),
B rows copied in pieces, all type pairs, new values on kept patterns. Every
entry against the oracle, and the structure against the level-by-level order."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.parity import compare_full

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def g():
    from paper_2607_22866_amd import gmagnus

    gmagnus.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return gmagnus


def _product(g, A, B, it=torch.int32, vt=torch.float64, path=None, **opts):
    dA, dB = (g.DeviceCSR.from_host(m, index_dtype=it, value_dtype=vt) for m in (A, B))
    with g.Plan(dA, dB, **opts) as p:
        rp, _ = p.symbolic()
        col, val = p.numeric()
        info = p.info()
    torch.cuda.synchronize()
    assert info.check_flags == 0 and info.n_heavy_rows > 0
    if path:
        assert g.PATH_NAMES[info.expansion_path] == path
    return rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()


# (A rows, inner size, columns, A entries per row, B entries per row)
SIZES = [
    (9, 300, 16383, 40, 200),     # one chunk, not full
    (9, 300, 16384, 40, 200),     # exactly one chunk
    (9, 300, 16385, 40, 200),     # one column in a second chunk
    (5, 40, 300, 30, 290),        # fewer columns than a wave's words
    (9, 300, 3 * 16384 + 5, 250, 40),      # regions of about 3300 products
    (9, 400, 40000, 200, 900),    # dense: over 7168 distinct columns a chunk
    (9, 300, 32768, 280, 1000),   # more long parts than the shared list holds
    (9, 50, 70000, 6, 20000),     # B rows copied in pieces, parts of thousands
    # regions of 4, 8 and 16 merged chunks, and of both sizes of group
    (12, 250, 17 * 16384, 60, 100),
    (40, 100, 16 * 16384, 60, 64),
    (40, 100, 32 * 16384, 40, 96),
    (40, 100, 37 * 16384 - 3, 40, 111),
    # the lists' tiles of 8, 16, 32 and 64 chunks (16: also the most chunks whose
    # lists are adjacent): full, and a chunk past it
    (9, 300, 8 * 16384, 200, 64),
    (9, 300, 8 * 16384 + 1, 200, 64),
    (9, 300, 16 * 16384, 150, 100),
    (9, 300, 16 * 16384 + 1, 150, 100),
    (9, 300, 32 * 16384, 100, 200),
    (9, 300, 32 * 16384 + 1, 100, 200),
    (9, 300, 64 * 16384, 100, 400),
    (9, 300, 64 * 16384 + 1, 100, 400),
    # regions of up to 2048 and up to 4096 distinct columns: the most that are
    # summed by 16-wave groups, and one more
    (512, 300, 2000, 60, 60),
    (513, 300, 2000, 60, 60),
    (512, 300, 3500, 60, 60),
    (513, 300, 3500, 60, 60),
]
DENSE, LONG_PARTS, MERGED = SIZES[5], SIZES[6], SIZES[10]


@pytest.mark.parametrize("m,k,n,a_d,b_d", SIZES)
def test_sizes(g, m, k, n, a_d, b_d):
    A, B = wl.erdos_renyi(m, k, a_d, 11), wl.erdos_renyi(k, n, b_d, 12)
    ref = oracle.spgemm(A, B)
    rp, col, val = _product(g, A, B, path="copy")
    compare_full(rp, col, val, ref)
    rp2, col2, _ = _product(g, A, B, flags=g.FLAG_LEVEL_BY_LEVEL)
    assert np.array_equal(rp, rp2) and np.array_equal(col, col2)


@pytest.mark.parametrize("it,vt", [(torch.int32, torch.float32), (torch.int64, torch.float64),
                                   (torch.int64, torch.float32)])
@pytest.mark.parametrize("m,k,n,a_d,b_d", [DENSE, LONG_PARTS, MERGED])
def test_types(g, it, vt, m, k, n, a_d, b_d):
    if it == torch.int32 and vt == torch.float32:
        n = min(n, 1 << 18)  # (fp32 values with int32 columns: one multisplit level at most)
    A, B = wl.erdos_renyi(m, k, a_d, 21), wl.erdos_renyi(k, n, b_d, 22)
    f32 = vt == torch.float32
    if f32:
        A, B = (x.with_values(x.val.astype(np.float32).astype(np.float64)) for x in (A, B))
    compare_full(*_product(g, A, B, it, vt, path="copy"), oracle.spgemm(A, B), f32=f32)


@pytest.mark.parametrize("m,k,n,a_d,b_d,path", [
    (7, 300, 16384, 250, 200, "rows"),  # fewer than 8 uniform rows
    (8, 300, 16384, 250, 200, "copy"),
    (7, 300, 8192, 250, 200, "copy"),   # ... but without a level
    (9, 300, 64 * 16384, 150, 30, "rows_two_level"),     # fewer products than (entry, chunk) pairs
    (9, 100, 256 * 16384, 100, 512, "rows_two_level"),   # 2 products a pair of uniform rows on 256 chunks
    (9, 100, 256 * 16384, 100, 1024, "copy"),            # 4 products a pair
    (40, 100, 256 * 16384, 20, 560, "copy"),             # 2.2 products a pair, small first-level chunks
])
def test_rule(g, m, k, n, a_d, b_d, path):
    # uniform rows on both sides of each line of the rule
    A, B = wl.erdos_renyi(m, k, a_d, 41), wl.erdos_renyi(k, n, b_d, 42)
    compare_full(*_product(g, A, B, path=path), oracle.spgemm(A, B))


# (memory next to what the rule admits: most of it the copy, the lists, the regions)
@pytest.mark.parametrize("m,k,n,a_d,b_d", [(9, 2000, 16384, 40, 200), (40, 100, 32 * 16384, 100, 46),
                                           (40, 100, 256 * 16384, 20, 560), DENSE])
@pytest.mark.parametrize("flags", [0, 256], ids=["", "keep_pattern"])
def test_memory(g, m, k, n, a_d, b_d, flags):
    # a workspace limit that the expansion of the same product keeps to is no
    # hindrance, nor is the copy's own peak; below it the call fails cleanly
    A, B = wl.erdos_renyi(m, k, a_d, 51), wl.erdos_renyi(k, n, b_d, 52)
    dA, dB = g.DeviceCSR.from_host(A), g.DeviceCSR.from_host(B)

    def peak(path, **opts):
        with g.Plan(dA, dB, flags=flags, **opts) as p:
            p.symbolic()
            p.numeric()
            info = p.info()
        assert info.check_flags == 0 and (g.PATH_NAMES[info.expansion_path] == "copy") == (path == "copy")
        return info.workspace_peak_bytes

    mine, other = peak("copy"), peak("expansion", dense_width_log2=13)
    assert mine <= other
    for limit in (other, mine):
        assert peak("copy", workspace_limit_bytes=limit) <= limit
    with pytest.raises(g.GmagnusError) as e:
        peak("copy", workspace_limit_bytes=mine // 4)
    assert e.value.status == 3 and "workspace limit" in str(e.value)
    assert peak("copy") == mine


def test_bytes_are_compulsory(g):
    # the copy and the lists are counted once, not once a product
    m, k, n, a_d, b_d = DENSE
    A, B = wl.erdos_renyi(m, k, a_d, 53), wl.erdos_renyi(k, n, b_d, 54)
    dA, dB = g.DeviceCSR.from_host(A), g.DeviceCSR.from_host(B)
    with g.Plan(dA, dB) as p:
        _, nnz = p.symbolic()
        p.numeric()
        info = p.info()
    assert g.PATH_NAMES[info.expansion_path] == "copy"
    parts = np.array([np.unique(r >> 14).size for r in np.split(B.col, B.row_ptr[1:-1])])
    used = np.unique(A.col)
    elems, segs = b_d * used.size, int(parts[A.col].sum())
    by = {name: info.kernel_bytes[i] for i, name in enumerate(g.K_NAMES)}
    assert by["chunk_symbolic"] == 2 * elems + 8 * segs
    assert by["chunk_numeric"] == 10 * elems + 12 * segs + 8 * A.nnz + 12 * nnz
    assert by["expand"] == 22 * elems + 4 * 3 * used.size


@pytest.mark.parametrize("it,vt", [(torch.int32, torch.float64), (torch.int64, torch.float32)])
def test_rows_copied_in_pieces(g, it, vt):
    # B rows around whole pieces of 2048 elements, in no order of length (an
    # empty one among them), over three chunks
    lens = [2049, 1, 2048, 4097, 0, 2047, 4096, 6145, 64, 4095, 12289]
    n = 40_000
    rng = np.random.default_rng(31)
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lens]
    rp = np.concatenate([[0], np.cumsum(lens)])
    B = wl.CSR(len(lens), n, rp.astype(np.int64), np.concatenate(cols).astype(np.int32), rng.random(int(rp[-1])))
    A = wl.uniform(24, len(lens), 0.8, 32)
    f32 = vt == torch.float32
    if f32:
        A, B = (x.with_values(x.val.astype(np.float32).astype(np.float64)) for x in (A, B))
    compare_full(*_product(g, A, B, it, vt, path="copy"), oracle.spgemm(A, B), f32=f32)


@pytest.mark.parametrize("seed,skew", [(5, (0.57, 0.19, 0.19)), (6, (0.7, 0.12, 0.12))])
def test_rmat_panel_and_new_values(g, seed, skew):
    # R-MAT rows (a few entries hold most products) over 8 chunks, empty B
    # rows among them; a row panel, then new values on the kept pattern
    A = wl.rmat(17, 2, *skew, seed)
    ip = oracle.row_products(A, A)
    r1 = int(np.searchsorted(np.cumsum(ip), 3_000_000)) + 1
    dA = g.DeviceCSR.from_host(A)
    rng = np.random.default_rng(seed)
    A2 = A.with_values(rng.uniform(-1.0, 1.0, A.nnz))
    with g.Plan(dA, dA, row_end=r1, flags=g.FLAG_KEEP_PATTERN | g.FLAG_CONCURRENT_STREAMS) as p:
        rp, _ = p.symbolic()
        for X in (A, A2):
            if X is A2:
                p.update_values(torch.from_numpy(A2.val).cuda())
            col, val = p.numeric()
            assert p.info().check_flags == 0 and g.PATH_NAMES[p.info().expansion_path] == "copy"
            compare_full(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(),
                         oracle.spgemm(X, X, rows=np.arange(r1)))
