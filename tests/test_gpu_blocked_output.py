"""The blocked decode's outputs at densities whose groups of 2048 parameters hold
fewer and more members than a wave's staging slots, with a partial last group,
and into views off the 16-byte grid.  Whole numbers: exact in both types."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vtype", ["i32", "f32"])
@pytest.mark.parametrize("density", [0.003, 0.06, 0.16, 0.3, 0.6])
def test_blocked_outputs(density, vtype):
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vt = torch.int32 if vtype == "i32" else torch.float32
    n = 3_000_017
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(density * 1000))
    x = torch.randint(1, 300, (n,), device="cuda", generator=gen)
    x = torch.where(torch.rand(n, device="cuda", generator=gen) < density, x, torch.zeros_like(x)).to(vt)
    # denser stretches: groups on both sides of the slots in one sketch
    x[100_000:101_500] = 5
    m = int((x != 0).sum())
    p = hc.hc_geometry_blocked(n, m, 1.6, 1024, 0, 9, vtype)
    y = torch.empty(p.cells, dtype=vt, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    for off in (0, 1):
        buf = torch.full((n + off,), 7, dtype=vt, device="cuda")
        mask = torch.full((p.words,), -1, dtype=torch.int32, device="cuda")
        ci = torch.full((m,), -1, dtype=torch.int32, device="cuda")
        cv = torch.zeros(m, dtype=vt, device="cuda")
        info = hc.alloc_info()
        hc.hc_decode(p, y, b, info, hc.alloc_workspace(p), x_out=buf[off:], mask=mask, coo_idx=ci,
                     coo_val=cv)
        inf = hc.read_info(info)
        assert (inf.n_support, inf.status) == (m, 0)
        assert torch.equal(ci.long(), torch.nonzero(x).reshape(-1))
        rec = ((mask[:, None] >> torch.arange(32, device="cuda")) & 1).reshape(-1)[:n].bool()
        assert int(rec.sum()) == inf.n_recovered
        assert not (rec & (x == 0)).any()
        assert inf.n_recovered >= 0.9 * m  # nearly every block peels at 1.6 cells per member
        assert torch.equal(buf[off:][rec], x[rec])
        assert not buf[off:][x == 0].any()
        assert torch.equal(cv, buf[off:][x != 0])
