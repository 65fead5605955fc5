"""Row products and column spans of the setup phase where its short cuts could
go wrong: rows inside, at the edge of and across a work group's entries, more
rows than it keeps in LDS, mostly wide B rows (one byte a row) with narrow and
long ones among them. The counts and every entry of C against the oracle."""
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


def csr(rows, n_cols, seed):
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    col = np.concatenate([np.asarray(r, np.int64) for r in rows])
    return wl.CSR(len(rows), n_cols, rp, col, np.random.default_rng(seed).uniform(-1.0, 1.0, col.size))


def wide_and_narrow(n_cols, seed):
    """1200 B rows: most span at least a quarter of the columns, every 16th 30 columns, one in 200 has 300 elements, some are empty."""
    rng = np.random.default_rng(seed)
    rows = []
    for k in range(1200):
        if k % 16 == 3:
            lo = int(rng.integers(0, n_cols - 30))
            rows.append(np.unique(lo + rng.integers(0, 30, 6)))
        elif k % 100 == 50:
            rows.append([])
        else:
            m = 300 if k % 200 == 7 else 5
            rows.append(np.unique(np.concatenate([[k % 50, n_cols - 1 - k % 70], rng.integers(0, n_cols, m)])))
    return csr(rows, n_cols, seed)


@pytest.mark.parametrize("n_cols", [65535, 65536, 300_007])
@pytest.mark.parametrize("it", [torch.int32, torch.int64])
def test_wide_rows(g, n_cols, it):
    rng = np.random.default_rng(1)
    B = wide_and_narrow(n_cols, 2)
    narrow = np.arange(3, 1200, 16)
    rows = [[int(rng.choice(narrow))] if i % 3 == 0 else  # fits a window
            np.unique(rng.integers(0, 1200, 1 + i % 40)) for i in range(1500)]
    A = csr(rows, 1200, 3)
    dA, dB = (g.DeviceCSR.from_host(m, index_dtype=it) for m in (A, B))
    assert np.array_equal(g.row_products(dA, dB).cpu().numpy(), oracle.row_products(A, B))
    rp, col, val = g.spgemm(dA, dB)
    compare_full(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(), oracle.spgemm(A, B))


@pytest.mark.parametrize("per_row", [1, 2, 3, 2047, 2048, 2049])
def test_rows_and_groups(g, per_row):
    # one entry a row (more rows than a work group keeps) up to rows as long as its entries
    n = 6000 if per_row < 4 else 7
    B = wide_and_narrow(70_000, 4)
    B = csr([B.col[a:b][:2] for _ in range(2) for a, b in zip(B.row_ptr[:-1], B.row_ptr[1:])], 70_000, 5)
    A = wl.erdos_renyi(n, 2400, min(per_row, 2400), 6)
    dA, dB = (g.DeviceCSR.from_host(m) for m in (A, B))
    ip = oracle.row_products(A, B)
    assert np.array_equal(g.row_products(dA, dB).cpu().numpy(), ip)
    for r0, r1 in ((0, n), (n // 3, n - 1)):
        with g.Plan(dA, dB, row_begin=r0, row_end=r1) as p:
            rp, _ = p.symbolic()
            col, val = p.numeric()
            info = p.info()
        assert info.check_flags == 0 and info.products_total == int(ip[r0:r1].sum())
        compare_full(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(),
                     oracle.spgemm(A, B, rows=np.arange(r0, r1)))
