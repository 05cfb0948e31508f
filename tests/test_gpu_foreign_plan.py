"""Decodes given a plan built for another geometry, on every kernel that reads
one past the size the whole-sketch decode takes: status 3, nothing peeled,
every member the median estimate from the aggregate.  The plans differ in seed
alone, or are for far smaller or larger geometries: only the header of such a
plan is known to exist, so nothing else of it may be read."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# (n, rows, vtype, density, support bound): the kernel that takes the plan
@pytest.mark.parametrize("n,rows,vtype,density,bound", [
    (1_300_007, 9, "i32", 0.004, "tight"),      # workgroups sharing a row's entries
    (1_300_007, 9, "f32", 0.004, "tight"),      # ... outputs zeroed beside the peel
    (1_300_007, 9, "i32", 0.004, "n"),          # ... outputs written by the emit
    (20_000_003, 1100, "i32", 0.03, "tight"),   # a workgroup per row
    (1_300_007, 500, "i32", 0.1, "tight"),      # a wave per row of few entries
    (1_300_007, 500, "f32", 0.1, "tight"),
    (5_000_011, 2100, "f32", 0.1, "tight"),     # a wave per row, rows to spare
    (5_000_011, 2100, "i32", 0.1, "n"),         # ... fewer cells than the bound
    (20_000_003, 2100, "i32", 0.05, "tight"),   # round 0 by rows
    (5_000_011, 2100, "i32", 0.3, "tight"),     # ... over dense batches
])
def test_foreign_plan(n, rows, vtype, density, bound):
    import torch
    import oracle
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vt = torch.int32 if vtype == "i32" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    x = torch.randint(1, 300, (n,), device="cuda", generator=gen)
    x = torch.where(torch.rand(n, device="cuda", generator=gen) < density, x, torch.zeros_like(x)).to(vt)
    m = int((x != 0).sum())
    seed = 41
    p = hc.make_params(n, rows, seed, 1024, vtype)
    y = torch.empty(p.cells, dtype=vt, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)

    def decode(cap, plan):
        out = torch.full((n,), 7, dtype=vt, device="cuda")
        mask = torch.full((p.words,), -1, dtype=torch.int32, device="cuda")
        ci = torch.full((m,), -1, dtype=torch.int32, device="cuda")
        cv = torch.zeros(m, dtype=vt, device="cuda")
        info = hc.alloc_info()
        hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, cap), x_out=out, mask=mask, coo_idx=ci,
                     coo_val=cv, max_support=cap, plan=plan)
        return out, mask, ci, cv, hc.read_info(info)

    # nothing peeled for another reason, without a plan
    ref = decode(m - 1, None)
    assert (ref[4].status, ref[4].n_recovered) == (1, 0)
    g = oracle.Geom(n=n, rows=rows, seed=seed, c=1024)
    sup = torch.nonzero(x).reshape(-1)
    some = sup[::max(1, m // 200)].cpu().numpy()
    if vtype == "i32":
        yh = y.cpu().numpy()
        est = np.array([oracle.query(g, yh, int(k)) for k in some], np.int32)
        assert np.array_equal(ref[0].cpu().numpy()[some], est)

    cap = {"tight": m, "n": 0}[bound]
    for other in (hc.make_params(n, rows, seed + 1, 1024, vtype),     # the same layout
                  hc.make_params(1000, 3, seed, 1024, vtype),         # 3 rows, 3 entries
                  hc.make_params(n, rows, seed, 256, vtype),
                  hc.make_params(n - 1, rows, seed, 1024, vtype),
                  hc.make_params(4 * n, rows + 1, seed, 1024, vtype)):
        got = decode(cap, hc.make_plan(other))
        assert got[4] == hc.DecodeInfo(m, 0, 0, 0, 3), got[4]
        assert not got[1].any()
        for a, e in zip(got[:4], ref[:4]):
            assert torch.equal(a, e)
        assert torch.equal(got[2].long(), sup)
