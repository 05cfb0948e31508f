"""Decodes over their own inputs, by a caller done with the aggregate: the
recovered mask into the aggregated bitmap, the dense sum into the buffer whose
head holds the aggregated sketch.  Sizes on both sides of the whole-sketch
decode, of the supports whose outputs are zeroed beside the peel and of the
bitmaps whose emit chunks are shared; outputs and summary are those of the
decode into buffers of their own."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vtype", ["i32", "f32"])
@pytest.mark.parametrize("gamma", [1.5, 0.95])  # everything peels; most of it is left
@pytest.mark.parametrize("n,density", [
    (300_007, 0.01),      # one launch
    (3_000_011, 0.005),   # zeroed beside the peel
    (3_000_011, 0.05),    # shared emit chunks
    (40_000_003, 0.03),
])
def test_decode_in_place(n, density, gamma, vtype):
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vt = torch.int32 if vtype == "i32" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    x = torch.randint(1, 300, (n,), device="cuda", generator=gen)
    x = torch.where(torch.rand(n, device="cuda", generator=gen) < density, x, torch.zeros_like(x)).to(vt)
    m = int((x != 0).sum())
    p = hc.hc_geometry(n, m, gamma, 1024, 23, vtype)
    y = torch.empty(p.cells, dtype=vt, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    ws = hc.alloc_workspace(p, m)
    info = hc.alloc_info()

    def decode(plan, ya, ba, out, mask):
        hc.hc_decode(p, ya, ba, info, ws, x_out=out, mask=mask, max_support=m, plan=plan)
        return out, mask, hc.read_info(info)

    for plan in (hc.make_plan(p), None):
        want = decode(plan, y, b, torch.empty_like(x), torch.empty_like(b))
        assert want[2].success == (gamma > 1)
        over = b.clone()
        got = [decode(plan, y, over, torch.empty_like(x), over)]
        if gamma > 1:  # estimates of what is left read the sketch to the end
            buf = torch.zeros_like(x)
            buf[:p.cells] = y
            got.append(decode(plan, buf[:p.cells], b, buf, torch.empty_like(b)))
        for g in got:
            assert g[2] == want[2]
            assert torch.equal(g[0], want[0]) and torch.equal(g[1], want[1])
