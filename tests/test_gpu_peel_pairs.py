"""The fp32 peel on both sides of the support size up to which its counters are
doubles updated beside their residuals (2^26 elements where 2^25 batches or more
leave no more bits, here one parameter each), and on sketches small
enough for every launch shape of the peel.

Values are whole numbers below 2^9 in magnitude, so every fp32 and fp64 sum on
the way is exact and the decode has to return the input bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,support,plan", [
    (1 << 27, 1 << 26, True),
    (1 << 27, (1 << 26) + 1, True),
    (1 << 27, 1 << 26, None),         # c = 1: the largest with doubles
    (1 << 27, (1 << 26) + 1, None),   # counters and residuals apart
    (3_000_001, 60_000, True),        # half the CUs
    (3_000_001, 60_000, False),
    (20_000_001, 1_390_000, True),    # just under 2^21 cells: half the CUs
    (20_000_001, 1_400_000, True),    # 2^21 to 2^23 cells: three quarters
    (40_000_003, 5_500_000, True),
    (40_000_003, 5_500_000, False),
    (40_000_003, 8_000_000, True),    # round 0 over the whole chip
    (40_000_003, 8_000_000, False),
])
def test_fp32_peel_returns_whole_numbers_exactly(n, support, plan):
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n % 1009 + support)
    x = torch.zeros(n, dtype=torch.float32, device="cuda")
    if 2 * support > n:  # every other parameter and one more
        idx = torch.cat([torch.arange(support - 1, device="cuda") * 2,
                         torch.tensor([1], device="cuda")])
    else:
        idx = torch.arange(support, device="cuda") * (n // support)
    v = torch.randint(1, 512, (support,), device="cuda", generator=gen).float()
    x[idx] = torch.where(torch.rand(support, device="cuda", generator=gen) < 0.5, -v, v)
    p = hc.hc_geometry(n, support, 1.5, 1 if plan is None else 1024, 77, "f32")
    y = torch.empty(p.cells, dtype=torch.float32, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    out = torch.empty_like(x)
    info = hc.alloc_info()
    ws = hc.alloc_workspace(p, support)
    hc.hc_decode(p, y, b, info, ws, x_out=out, max_support=support,
                 plan=hc.make_plan(p) if plan else None)
    inf = hc.read_info(info)
    assert (inf.success, inf.status, inf.n_support) == (1, 0, support), inf
    assert torch.equal(out, x)


@pytest.mark.parametrize("plan", [True, False])
@pytest.mark.parametrize("n,support,rows", [
    # past the short bitmaps: the cells per element from which pairs are kept (1.2,
    # below which not all of it peels), and from 0.4 of the parameters on up to
    # which (2.2 with a plan, 2 without)
    (10_000_000, 1_000_000, 1171), (10_000_000, 1_000_000, 1172),
    (6_000_000, 2_400_000, 5156), (6_000_000, 2_400_000, 5157), (6_000_000, 2_399_999, 5157),
    (6_000_000, 3_000_000, 5859), (6_000_000, 3_000_000, 5860),
])
def test_fp32_pairs_by_cells_per_element(n, support, rows, plan):
    """Against the int32 decode of the same whole numbers, every output."""
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    idx = torch.randperm(n, device="cuda", generator=gen)[:support]
    v = torch.randint(1, 300, (support,), device="cuda", generator=gen, dtype=torch.int32)
    got = []
    for vt, name in ((torch.float32, "f32"), (torch.int32, "i32")):
        x = torch.zeros(n, dtype=vt, device="cuda")
        x[idx] = v.to(vt)
        p = hc.make_params(n, rows, 3, 1024, name)
        y = torch.empty(p.cells, dtype=vt, device="cuda")
        b = torch.empty(p.words, dtype=torch.int32, device="cuda")
        hc.hc_encode(p, x, y, b)
        for cap in (support, 0):
            out = torch.full((n,), 7, dtype=vt, device="cuda")
            mask = torch.full((p.words,), -1, dtype=torch.int32, device="cuda")
            info = hc.alloc_info()
            hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, cap), x_out=out, mask=mask,
                         max_support=cap, plan=hc.make_plan(p) if plan and vt is torch.float32 else None)
            got.append((out.double(), mask, hc.read_info(info)))
    for g in got[:-1]:
        assert g[2] == got[-1][2]
        assert torch.equal(g[1], got[-1][1]) and torch.equal(g[0], got[-1][0])
