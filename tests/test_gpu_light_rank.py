"""Light rows summed by rank, at the sizes where it can go wrong: product
counts around the bins' limits, column spans that need one to five levels of
words, rows whose entries outnumber their products (empty B rows) or meet one
long B row, all type pairs. Every entry against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.parity import compare_full

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NO_WINDOW = 4


@pytest.fixture(scope="module")
def g():
    from paper_2607_22866_amd import gmagnus

    gmagnus.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return gmagnus


def check(g, A, B, it=torch.int32, vt=torch.float64):
    f32 = vt == torch.float32
    if f32:
        A, B = (x.with_values(x.val.astype(np.float32).astype(np.float64)) for x in (A, B))
    dA, dB = (g.DeviceCSR.from_host(m, index_dtype=it, value_dtype=vt) for m in (A, B))
    with g.Plan(dA, dB, flags=NO_WINDOW) as p:
        rp, _ = p.symbolic()
        col, val = p.numeric()
        info = p.info()
    torch.cuda.synchronize()
    assert info.check_flags == 0 and info.n_heavy_rows == 0
    compare_full(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(), oracle.spgemm(A, B), f32=f32)


def ragged(lens, n_cols, seed):
    """CSR with lens[i] distinct random columns in row i."""
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n_cols, size=int(x), replace=False)) for x in lens]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate(cols).astype(np.int32) if rp[-1] else np.zeros(0, np.int32)
    return wl.CSR(len(lens), n_cols, rp, col, rng.uniform(-1.0, 1.0, int(rp[-1])))


@pytest.mark.parametrize("it,vt", [(torch.int32, torch.float64), (torch.int64, torch.float32)])
def test_product_counts(g, it, vt):
    # row i of A meets B rows of 1, 2, 4, ... elements: every product count
    # around the bins' limits (256, 512, 1024, 2048, 3456)
    counts = sorted({c + d for c in (2, 64, 256, 512, 1024, 2048) for d in (-1, 0, 1)} | {3455, 3456})
    B = ragged([1 << b for b in range(12)], 5000, 3)
    bits = [[b for b in range(12) if c >> b & 1] for c in counts]
    rp = np.concatenate([[0], np.cumsum([len(x) for x in bits])]).astype(np.int64)
    col = np.concatenate(bits).astype(np.int32)
    A = wl.CSR(len(bits), 12, rp, col, np.random.default_rng(4).uniform(-1.0, 1.0, col.size))
    check(g, A, B, it, vt)


@pytest.mark.parametrize("log2", [5, 10, 13, 17, 18, 19, 22, 23, 24, 28, 30])
@pytest.mark.parametrize("per_row", [3, 24, 50])
def test_column_spans(g, log2, per_row):
    # 9, 576 and 2500 products over 2^log2 columns (and one more)
    for n in ((1 << log2), (1 << log2) + 1):
        d = min(per_row, 1 << log2)
        A, B = wl.erdos_renyi(40, 200, per_row, 5), wl.wide(200, n, d, 6)
        check(g, A, B, torch.int64 if log2 >= 24 else torch.int32)


def test_empty_and_long_parts(g):
    # 3000 entries, all but a few into empty B rows; and one B row of 3456 elements
    lens = np.zeros(4000, np.int64)
    lens[::97] = 40
    lens[1] = 3456
    B = ragged(lens, 100000, 7)
    dense = ragged([3000, 2999, 130], 4000, 8)
    dense = wl.CSR(3, 4000, dense.row_ptr, np.where(dense.col == 1, 2, dense.col).astype(np.int32), dense.val)
    # (columns stay distinct: column 1 is dropped by rebuilding each row)
    rows = [np.unique(dense.col[a:b]) for a, b in zip(dense.row_ptr[:-1], dense.row_ptr[1:])] + [np.array([1], np.int32)]
    rp = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    A = wl.CSR(4, 4000, rp, col, np.random.default_rng(9).uniform(-1.0, 1.0, col.size))
    check(g, A, B)


@pytest.mark.parametrize("per_row", [20, 40, 41, 60, 69])
@pytest.mark.parametrize("distinct", [50, 51, 300])
def test_many_repeats(g, per_row, distinct):
    # rows of 1000, 2000, 2050, 3000 and 3450 products that meet `distinct` columns
    # spread over 2^20, up to 69 times each
    rng = np.random.default_rng(12)
    pool = np.sort(rng.choice(1 << 20, distinct, replace=False)).astype(np.int32)
    cols = [pool[np.sort(rng.choice(distinct, 50, replace=False))] for _ in range(80)]
    B = wl.CSR(80, 1 << 20, np.arange(81, dtype=np.int64) * 50, np.concatenate(cols), rng.uniform(-1.0, 1.0, 4000))
    check(g, wl.erdos_renyi(30, 80, per_row, 13), B)


def test_more_rows_than_one_launch(g):
    # 2^22 light rows and three more, of two products each
    m = (1 << 22) + 3
    rng = np.random.default_rng(14)
    A = wl.CSR(m, 1000, np.arange(m + 1, dtype=np.int64), rng.integers(0, 1000, m).astype(np.int32), rng.uniform(-1.0, 1.0, m))
    check(g, A, ragged(np.full(1000, 2), 1 << 20, 15))
