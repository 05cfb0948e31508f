"""Decodes whose dense outputs are zeroed beside the peel (a support bound of at
most one element per 64 parameters) against the decode of the same aggregate
with the loosest bound, which writes its outputs whole, and against the input:
support in runs and scattered, a chunk of 32,768 parameters denser than the
emit's window, lengths off every grid, each output alone, failures."""
import pytest

pytestmark = pytest.mark.gpu


def _make(n, kind, vt):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    m = n // 80
    if kind == "runs":
        start = torch.randint(0, n // 64, (m // 64,), device="cuda", generator=gen) * 64
        idx = (start[:, None] + torch.arange(64, device="cuda")).reshape(-1)
    elif kind == "cluster":  # one chunk with over 1024 members, the others sparse
        idx = torch.cat([torch.arange(40000, 43000, device="cuda"),
                         torch.randint(0, n, (m // 2,), device="cuda", generator=gen)])
    else:
        idx = torch.randint(0, n, (m,), device="cuda", generator=gen)
    idx = torch.unique(idx[idx < n])
    idx = torch.unique(torch.cat([idx, torch.tensor([0, n - 1], device="cuda")]))
    x = torch.zeros(n, dtype=vt, device="cuda")
    v = torch.randint(1, 400, (idx.numel(),), device="cuda", generator=gen)
    x[idx] = v.to(vt)
    return x, idx.numel()


def _decode(hc, p, y, b, support, outs, plan):
    import torch
    n, vt = int(p.n), y.dtype
    dev = "cuda"
    o = {}
    if "x" in outs:
        o["x_out"] = torch.full((n,), 7, dtype=vt, device=dev)
    if "mask" in outs:
        o["mask"] = torch.full((p.words,), -1, dtype=torch.int32, device=dev)
    if "coo" in outs:
        o["coo_idx"] = torch.full((max(support, 1),), -1, dtype=torch.int32, device=dev)
        o["coo_val"] = torch.zeros(max(support, 1), dtype=vt, device=dev)
    info = hc.alloc_info()
    hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, support), max_support=support, plan=plan, **o)
    return o, hc.read_info(info)


@pytest.mark.parametrize("vtype", ["i32", "f32"])
@pytest.mark.parametrize("n,kind", [(2_097_152 + 13, "spread"), (5_000_002, "runs"),
                                    (4_194_304, "cluster"), (1_500_003, "cluster")])
def test_filled_decode_matches(n, kind, vtype):
    import torch
    import paper_2402_07529_amd as hc
    vt = torch.int32 if vtype == "i32" else torch.float32
    x, m = _make(n, kind, vt)
    p = hc.hc_geometry(n, m, 1.35, 1024, 5, vtype)
    y = torch.empty(p.cells, dtype=vt, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    for plan in (None, hc.make_plan(p)):
        for outs in ("x mask coo", "x", "x mask", "x coo", "mask"):
            o, inf = _decode(hc, p, y, b, m, outs.split(), plan)
            assert (inf.success, inf.n_support) == (1, m)
            if "x_out" in o:  # whole numbers: exact in fp32 too
                bad = torch.nonzero(o["x_out"] != x).reshape(-1)
                assert bad.numel() == 0, (outs, bad.numel(), bad[:8], o["x_out"][bad[:8]], x[bad[:8]])
            if "mask" in o:
                assert torch.equal(o["mask"], b), outs
            if "coo_idx" in o:
                assert torch.equal(o["coo_idx"].long(), torch.nonzero(x).reshape(-1))
                assert torch.equal(o["coo_val"], x[x != 0])
        whole, winf = _decode(hc, p, y, b, n, ["x", "mask", "coo"], plan)  # written whole
        tight, inf = _decode(hc, p, y, b, m, ["x", "mask", "coo"], plan)
        assert winf == inf
        assert torch.equal(whole["x_out"], tight["x_out"]) and torch.equal(whole["mask"], tight["mask"])
        for k in ("coo_idx", "coo_val"):
            assert torch.equal(whole[k][:m], tight[k])


@pytest.mark.parametrize("gamma,short", [(1.0, 0), (1.35, 1)])
def test_filled_decode_failures(gamma, short):
    """A sketch too narrow to peel, and a support over the bound: the estimates
    and the mask of the decode that does not fill."""
    import torch
    import paper_2402_07529_amd as hc
    n = 3_000_001
    x, m = _make(n, "spread", torch.int32)
    p = hc.hc_geometry(n, m, gamma, 1024, 6, "i32")
    y = torch.empty(p.cells, dtype=torch.int32, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    plan = hc.make_plan(p)
    o, inf = _decode(hc, p, y, b, m - short, ["x", "mask", "coo"], plan)
    assert inf.success == 0 and inf.status == short
    # the reference: not filled, as its dense output is not 16-byte aligned
    out = torch.full((n + 1,), 7, dtype=torch.int32, device="cuda")
    mask = torch.full((p.words,), -1, dtype=torch.int32, device="cuda")
    info = hc.alloc_info()
    hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, m - short), x_out=out[1:], mask=mask,
                 max_support=m - short, plan=plan)
    assert hc.read_info(info) == inf
    assert torch.equal(o["x_out"], out[1:]) and torch.equal(o["mask"], mask)
    k = m - short
    assert torch.equal(o["coo_val"][:k], out[1:][o["coo_idx"][:k].long()])
