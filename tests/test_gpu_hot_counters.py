"""Counters of a cell whose members' positions sum to more than 2^32, in both
value types.  The support is dense batches that fill every row but a few, so
that nothing there can be peeled, and then one element of each of some batches
that land on one of the rows left out: all of them meet in that row's cell 0,
each but one with a further cell of its own.  Round 0 recovers those, which
leaves the last alone in the hot cell, and round 1 recovers it through that
cell only.  Values are whole numbers and every sum stays below 2^24, so fp32 is
exact too."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def hot_support(n, c, rows, free, nbulk, seed):
    """(ascending indices, the places of those to be peeled among them)."""
    nb = n // c
    g = oracle.Geom(n=n, rows=rows, seed=seed, c=c)
    cl, _ = oracle.cells(g, np.arange(nb, dtype=np.uint64) * c)
    r = (cl // c).astype(np.int64)
    bias = (cl % c).astype(np.int64)
    hot = free  # the hot row; rows 0 .. free - 1 are the peelable elements' own
    bulk = np.nonzero((r > hot).all(1))[0][:nbulk]
    assert bulk.size == nbulk
    late = np.arange(nb) > bulk[-1]
    b, j = np.nonzero((r == hot) & late[:, None])
    t = (0 - bias[b, j]) & (c - 1)  # the column that lands in the hot cell
    own = r[b] < free
    cell = r[b] * c + ((t[:, None] + bias[b]) & (c - 1))
    # cells in the free rows, one or two, that no other element has
    cells, count = np.unique(cell[own], return_counts=True)
    alone = np.isin(cell, cells[count == 1])
    pick = own.any(1) & (alone | ~own).all(1)
    last = np.nonzero(own.sum(1) == 0)[0][0]  # both other cells among the bulk's
    e = np.concatenate([b[pick] * c + t[pick], [b[last] * c + t[last]]])
    idx = np.concatenate([(bulk[:, None] * c + np.arange(c)).reshape(-1), np.sort(e)])
    return idx, np.arange(nbulk * c, idx.size)


@pytest.mark.parametrize("vtype", ["f32", "i32"])
@pytest.mark.parametrize("n,c,rows,free,support", [
    # 1.2 cells per element or more: fp32 counters are doubles beside the residuals
    (1 << 31, 1024, 900, 720, 750_000),      # two workgroups to a row
    (1 << 31, 1024, 1300, 1040, 1_080_000),  # a workgroup per row
    (1 << 31, 256, 5000, 4000, 1_030_000),   # a wave per row
    # far fewer cells: fp32 counters and residuals in arrays of their own
    (1 << 28, 1024, 1000, 100, 1 << 26),
    (1 << 29, 1024, 2000, 200, 1 << 26),
    (1 << 28, 256, 4096, 409, (1 << 26) + 12_000),
])
def test_hot_cell(n, c, rows, free, support, vtype):
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    seed = 91
    idx, hot = hot_support(n, c, rows, free, (support - 8000) // c, seed)
    m = idx.size
    assert m <= support and (5 * rows * c >= 6 * m) == (support < 1 << 26)
    assert int(hot.sum()) >= 2**32  # the hot cell's positions
    print(f"n={n} c={c} rows={rows} support={m} hot={hot.size} {vtype}", flush=True)
    vt = torch.int32 if vtype == "i32" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c + rows)
    val = torch.randint(1, 512, (m,), device="cuda", generator=gen).to(vt)
    di = torch.from_numpy(idx.astype(np.int32)).cuda()
    p = hc.make_params(n, rows, seed, c, vtype)
    y = torch.empty(p.cells, dtype=vt, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode_coo(p, di, val, y, b)
    mask = torch.empty(p.words, dtype=torch.int32, device="cuda")
    ci, cv = torch.empty_like(di), torch.empty_like(val)
    info = hc.alloc_info()
    ws = hc.alloc_workspace(p, m)
    want = np.zeros(p.words, np.uint32)
    np.bitwise_or.at(want, idx[hot] >> 5, np.uint32(1) << (idx[hot] & 31).astype(np.uint32))
    for plan in (hc.make_plan(p), None):
        hc.hc_decode(p, y, b, info, ws, mask=mask, coo_idx=ci, coo_val=cv, max_support=m, plan=plan)
        inf = hc.read_info(info)
        assert (inf.n_support, inf.n_recovered, inf.rounds, inf.status) == (m, hot.size, 2, 0), inf
        assert np.array_equal(mask.cpu().numpy().view(np.uint32), want)
        assert torch.equal(ci, di) and torch.equal(cv[hot[0]:], val[hot[0]:])
