"""GPU parity of the single-launch paths of small global sketches, on both
sides of the bounds that select them: the row-gathering encode (at most 1024
batches and rows, c >= 256) and the decode whose workgroups each peel the
whole sketch in LDS (at most 1024 batches, the cells in one workgroup's LDS).

Bar: int32 bit-exact against the oracle, every output; fp32 structure exact
and values within the derived bounds of test_gpu_parity."""
import numpy as np
import pytest

import workloads as wl
from hc_pipeline import gpu_run, oracle_run
from test_gpu_parity import assert_same_info, check_fp32, check_int

pytestmark = pytest.mark.gpu


def _w(n, vtype="i32", W=3, density=0.01):
    return wl.make("synthetic", vtype, n=n, W=W, density=density, overlap=0.5, data_seed=n % 97,
                   hash_seed=n % 89)


# batches: 1, 2, 64, 1024 (the last that fits), 1025 (the general paths); rows
# 3 (columns split over workgroups, the list over waves), 14 and 15 (14 rows of
# 1024 is the largest int32 sketch whose decode fits LDS beside 1024 batches)
@pytest.mark.parametrize("n,rows,c", [
    (1024, 3, 1024), (1025, 3, 1024), (65536 + 7, 5, 1024), (1024 * 1024, 14, 1024),
    (1024 * 1024, 15, 1024), (1024 * 1024 + 1, 14, 1024), (700 * 1024 + 33, 9, 1024),
    (512 * 1024, 28, 512), (256 * 1024, 56, 256), (256 * 1024 + 1, 40, 256), (1024 * 32, 100, 32),
    (640 * 1024, 15, 1024), (640 * 1024 + 1, 15, 1024),  # 15 rows fit beside 640 batches
])
def test_small_int32(n, rows, c):
    check_int(_w(n, density=min(0.3, 0.25 * rows * c / n)), rows, c, use_plan=c >= 256)


# fp32: 10 rows fit beside 1024 batches, 11 beside 347
@pytest.mark.parametrize("n,rows", [
    (300 * 1024 + 5, 10), (300 * 1024 + 5, 11), (1024 * 1024, 9), (1024 * 1024, 10),
    (1024 * 1024, 11), (300 * 1024 + 5, 12), (347 * 1024, 11), (347 * 1024 + 1, 11),
])
def test_small_fp32(n, rows):
    check_fp32(_w(n, "f32", density=min(0.3, 0.25 * rows * 1024 / n)), rows, 1024)


# more rows than batches to share out (no column split) and the row bound
@pytest.mark.parametrize("rows", [256, 1024, 1025])
def test_small_encode_many_rows(rows):
    w = _w(90 * 1024 + 3, density=0.3, W=2)
    check_int(w, rows, 1024)


def test_small_decode_reports_overflow_and_foreign_plan():
    import paper_2402_07529_amd as hc
    w = _w(200 * 1024 + 9)
    rows = 12
    ref = oracle_run(w, rows, 1024)
    g = gpu_run(w, rows, 1024, max_support=w.n_agg - 1)
    assert (g["info"].status, g["info"].success, g["info"].n_recovered) == (1, 0, 0)
    assert g["info"].n_support == w.n_agg and not g["mask"].any()
    other = hc.make_plan(hc.make_params(w.n, rows, w.hash_seed + 1, 1024, w.vtype))
    f = gpu_run(w, rows, 1024, plan=other)
    assert (f["info"].status, f["info"].success, f["info"].n_support) == (3, 0, w.n_agg)
    assert np.array_equal(g["x"], f["x"]) and not f["mask"].any()
    # at the bound itself everything is peeled
    h = gpu_run(w, rows, 1024, max_support=w.n_agg)
    assert_same_info(h["info"], ref["info"])
    assert np.array_equal(h["x"], ref["x"])


@pytest.mark.parametrize("vtype", ["i32", "f32"])
def test_small_unaligned_gradient_and_partial_coo(vtype):
    """A gradient off the 16-byte grid, a COO list shorter than the support."""
    import torch
    import paper_2402_07529_amd as hc
    w = _w(150 * 1024 + 11, vtype, W=1)
    p = hc.hc_geometry(w.n, w.n_agg, 1.4, 1024, w.hash_seed, vtype)
    vt = torch.int32 if vtype == "i32" else torch.float32
    buf = torch.zeros(w.n + 3, dtype=vt, device="cuda")
    x = buf[1:w.n + 1]
    x.copy_(torch.from_numpy(w.dense(0)))
    y = torch.empty(p.cells, dtype=vt, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    cap = w.n_agg // 2
    idx = torch.full((cap + 8,), -1, dtype=torch.int32, device="cuda")
    val = torch.zeros(cap + 8, dtype=vt, device="cuda")
    info = hc.alloc_info()
    hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, w.n_agg), coo_idx=idx[:cap],
                 coo_val=val[:cap], max_support=w.n_agg)
    inf = hc.read_info(info)
    assert inf.success == 1 and inf.n_support == w.n_agg
    assert np.array_equal(idx[:cap].cpu().numpy().view(np.uint32), w.idx[0][:cap])
    assert (idx[cap:] == -1).all() and (val[cap:] == 0).all()
    got, want = val[:cap].cpu().numpy(), w.val[0][:cap]
    # one worker: fp32 cells of few terms, peeled in fp64
    assert np.array_equal(got, want) if vtype == "i32" else \
        np.max(np.abs(got - want)) <= 1e-5 * np.max(np.abs(want))


# past the small paths, few long rows: several workgroups share a row's plan
# entries (c = 256, 512, 1024), and the bitmap's chunks are shared by the emit
@pytest.mark.parametrize("n,rows,c,density", [
    (1_300_007, 4, 1024, 0.0005), (1_300_007, 33, 1024, 0.006), (2_000_003, 7, 512, 0.0004),
    (1_100_001, 18, 256, 0.001), (4_194_304 + 1, 40, 1024, 0.003),
])
def test_few_long_rows_planned(n, rows, c, density):
    check_int(_w(n, W=2, density=density), rows, c, use_plan=True)
    check_int(_w(n, W=2, density=density), rows, c, use_plan=False)


@pytest.mark.parametrize("n,rows", [(1_300_007, 9), (4_194_304 + 1, 40)])
def test_few_long_rows_planned_fp32(n, rows):
    check_fp32(_w(n, "f32", W=2, density=0.2 * rows * 1024 / n), rows, 1024, use_plan=True)
