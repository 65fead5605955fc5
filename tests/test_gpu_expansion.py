"""The expansion of heavy rows in its derived shape (final chunks of 8192
columns), which the default rule takes for sparse, evenly spread or few rows
only: forced here by naming the derived width. One level and both levels in
one pass, every accumulator of final chunks (more dense chunks than work
groups, so that each of these goes from chunk to chunk), all type pairs, new
values on kept patterns. Every entry against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.parity import compare_full

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TYPES = [(torch.int32, torch.float64), (torch.int32, torch.float32), (torch.int64, torch.float64),
         (torch.int64, torch.float32)]
TYPE_IDS = ["i32-f64", "i32-f32", "i64-f64", "i64-f32"]
DERIVED = dict(dense_width_log2=13)


@pytest.fixture(scope="module")
def g():
    from paper_2607_22866_amd import gmagnus

    gmagnus.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return gmagnus


def rounded(M, vt):
    """The matrix the GPU sees: values rounded to fp32 when vt is float32."""
    return M.with_values(M.val.astype(np.float32).astype(np.float64)) if vt == torch.float32 else M


def check(g, A, B, it, vt, path, **opts):
    A, B = rounded(A, vt), rounded(B, vt)
    dA, dB = (g.DeviceCSR.from_host(m, index_dtype=it, value_dtype=vt) for m in (A, B))
    with g.Plan(dA, dB, **DERIVED, **opts) as p:
        rp, _ = p.symbolic()
        col, val = p.numeric()
        info = p.info()
    torch.cuda.synchronize()
    assert info.check_flags == 0 and info.params.dense_width == 8192
    assert g.PATH_NAMES[info.expansion_path] == path
    rows = np.arange(opts.get("row_begin", 0), opts.get("row_end", A.n_rows))
    compare_full(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(), oracle.spgemm(A, B, rows=rows),
                 f32=vt == torch.float32)
    return info


@pytest.mark.parametrize("it,vt", TYPES, ids=TYPE_IDS)
def test_more_dense_chunks_than_work_groups(g, it, vt):
    # 70 rows of about 6000 products in each of 8 final chunks
    A, B = wl.erdos_renyi(70, 300, 160, 61), wl.erdos_renyi(300, 65536, 300, 62)
    info = check(g, A, B, it, vt, "rows")
    assert info.n_leaves_dense == 560 and info.levels_run == 1


@pytest.mark.parametrize("it,vt", TYPES, ids=TYPE_IDS)
def test_one_level_rmat(g, it, vt):
    A = wl.rmat(17, 8, 0.57, 0.19, 0.19, 63)
    ip = oracle.row_products(A, A)
    info = check(g, A, A, it, vt, "rows", row_end=int(np.searchsorted(np.cumsum(ip), 3_000_000)) + 1)
    assert info.n_leaves_dense > 0 and info.n_leaves_rank > 0


@pytest.mark.parametrize("it,vt", [t for t in TYPES if t != (torch.int32, torch.float32)],
                         ids=[i for i in TYPE_IDS if i != "i32-f32"])
@pytest.mark.parametrize("scale", [19, 21])
def test_two_levels_rmat(g, it, vt, scale):
    # hub rows first; 2^14 and 2^16 columns a first-level chunk
    A = wl.rmat(scale, 4, 0.57, 0.19, 0.19, 64)
    ip = oracle.row_products(A, A)
    info = check(g, A, A, it, vt, "rows_two_level", row_end=int(np.searchsorted(np.cumsum(ip), 3_000_000)) + 1)
    assert info.levels_run == 2 and info.n_leaves_dense > 0 and info.n_leaves_rank > 0


@pytest.mark.parametrize("n", [65536, 1 << 19])
def test_new_values(g, n):
    A, B = wl.erdos_renyi(20, 300, 160, 65), wl.erdos_renyi(300, n, 300, 66)
    dA, dB = g.DeviceCSR.from_host(A), g.DeviceCSR.from_host(B)
    rng = np.random.default_rng(67)
    with g.Plan(dA, dB, flags=g.FLAG_KEEP_PATTERN, **DERIVED) as p:
        rp, _ = p.symbolic()
        for again in (False, True, True):
            if again:
                A, B = (m.with_values(rng.uniform(-1.0, 1.0, m.nnz)) for m in (A, B))
                p.update_values(torch.from_numpy(A.val).cuda(), torch.from_numpy(B.val).cuda())
            col, val = p.numeric()
            info = p.info()
            assert info.check_flags == 0 and g.PATH_NAMES[info.expansion_path].startswith("rows")
            compare_full(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(), oracle.spgemm(A, B))
