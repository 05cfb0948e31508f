"""Rounds by rows over batches on both sides of the quarter density at which a
batch is taken parameter by parameter: the decode with the plan against the one
without (counters by atomics, round 0 entry by entry) and against the input."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [256, 512, 1024])
@pytest.mark.parametrize("overfull", [False, True])
def test_dense_and_sparse_batches(c, overfull):
    import torch
    import paper_2402_07529_amd as hc
    n = 6000 * c + 37  # ragged last batch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c)
    nb = (n + c - 1) // c
    # members per batch: none, one, c/4 - 1, c/4, c/4 + 1, three quarters, all
    want = torch.tensor([0, 1, c // 4 - 1, c // 4, c // 4 + 1, 3 * c // 4, c], device="cuda")
    want = want[torch.arange(nb, device="cuda") % want.numel()]
    order = torch.rand((nb, c), device="cuda", generator=gen).argsort(1)
    x = (order < want[:, None]).reshape(-1)[:n].to(torch.int32)
    x *= torch.randint(-2**30, 2**30, (n,), device="cuda", generator=gen, dtype=torch.int32) | 1
    support = int((x != 0).sum())
    # at least eight rows per CU and a cell per element of the support bound,
    # so that rows are taken a wave each; at one cell per element most of the
    # support cannot be peeled
    p = hc.hc_geometry(n, support, 1.0 if overfull else 1.5, c, 11, "i32")
    assert int(p.rows) >= 2048 and p.cells >= support
    y = torch.empty(p.cells, dtype=torch.int32, device="cuda")
    b = torch.empty(p.words, dtype=torch.int32, device="cuda")
    hc.hc_encode(p, x, y, b)
    got = []
    for plan in (hc.make_plan(p), None):
        out = torch.full((n,), 7, dtype=torch.int32, device="cuda")
        mask = torch.full((p.words,), -1, dtype=torch.int32, device="cuda")
        info = hc.alloc_info()
        hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, support), x_out=out, mask=mask,
                     max_support=support, plan=plan)
        got.append((out, mask, info[:hc.INFO_BYTES].clone()))
    torch.cuda.synchronize()
    for a, e in zip(*got):
        assert torch.equal(a, e)
    if not overfull:
        assert torch.equal(got[0][0], x)
