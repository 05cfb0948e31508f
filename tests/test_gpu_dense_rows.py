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


def _hot_row_support(n, c, rows, seed, density, gen):
    """A random support of that density and, in every batch landing on the
    busiest row, the element that falls into the row's cell 0."""
    import numpy as np
    import torch
    import oracle
    nb = n // c
    g = oracle.Geom(n=n, rows=rows, seed=seed, c=c)
    cl, _ = oracle.cells(g, np.arange(nb, dtype=np.uint64) * c)
    r, bias = (cl // c).astype(np.int64), (cl % c).astype(np.int64)
    busiest = int(np.argmax(np.bincount(r.reshape(-1), minlength=rows)))
    b, j = np.nonzero(r == busiest)
    hot = torch.from_numpy(b * c + ((0 - bias[b, j]) & (c - 1))).cuda()
    member = torch.rand(n, device="cuda", generator=gen) < density
    member[hot] = True
    return member, hot


@pytest.mark.parametrize("c,rows", [(1024, 147456), (512, 294912), (256, 589824)])
def test_unpackable_dense_support(c, rows):
    """A support of half of 2^28 parameters in a sketch of 1.12 cells each,
    and a hot cell whose counter does not pack: the row passes keep counters
    and residuals apart, no further round goes by rows and the peel starts at
    round 1.  Against the decode without a plan: every output and the summary."""
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, seed = 1 << 28, 17
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c)
    member, hot = _hot_row_support(n, c, rows, seed, 0.503, gen)
    support = int(member.sum())
    assert support >= n // 2 and rows * c >= support
    kp = (support - 1).bit_length()
    pos = torch.cumsum(member, 0, dtype=torch.int64)[hot] - 1
    assert hot.numel() * 2**kp + int(pos.sum()) >= 2**32
    x = torch.randint(-2**30, 2**30, (n,), device="cuda", generator=gen, dtype=torch.int32) | 1
    x *= member
    p = hc.make_params(n, rows, seed, c, "i32")
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
        got.append((out, mask, hc.read_info(info)))
    assert got[0][2] == got[1][2] and 0 < got[0][2].n_recovered < support
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("c", [256, 512, 1024])
@pytest.mark.parametrize("gamma", [1.3, 1.5, 2.2])  # cells to spare from 1.4 on
@pytest.mark.parametrize("per_batch", [1 / 16, 1 / 3, 1 / 2])
def test_row_rounds_by_support(per_batch, gamma, c):
    """Supports on both sides of the densities from which further rounds go by
    rows, under a tight bound, one just below and at each density, and none:
    every decode is the one without a plan."""
    import torch
    import paper_2402_07529_amd as hc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 8192 * c
    gen = torch.Generator(device="cuda")
    gen.manual_seed(c)
    idx = torch.randperm(n, device="cuda", generator=gen)
    for support in (int(n * per_batch) - 1, int(n * per_batch) + 1):
        x = torch.zeros(n, dtype=torch.int32, device="cuda")
        x[idx[:support]] = torch.randint(-2**30, 2**30, (support,), device="cuda", generator=gen,
                                         dtype=torch.int32) | 1
        # enough rows to be taken a wave each, and a cell per element of every bound
        p = hc.make_params(n, max(8192, int(gamma * support) // c + 1), 5, c, "i32")
        plan = hc.make_plan(p)
        y = torch.empty(p.cells, dtype=torch.int32, device="cuda")
        b = torch.empty(p.words, dtype=torch.int32, device="cuda")
        hc.hc_encode(p, x, y, b)

        def decode(cap, plan):
            out = torch.full((n,), 7, dtype=torch.int32, device="cuda")
            mask = torch.full((p.words,), -1, dtype=torch.int32, device="cuda")
            info = hc.alloc_info()
            hc.hc_decode(p, y, b, info, hc.alloc_workspace(p, cap), x_out=out, mask=mask,
                         max_support=cap, plan=plan)
            return out, mask, hc.read_info(info)

        want = decode(support, None)
        assert want[2].success and torch.equal(want[0], x)
        for cap in (support, n // 3, n // 2 - 1, n // 2, n - 1, 0):
            if cap and cap < support:
                continue
            got = decode(cap, plan)
            assert got[2] == want[2], cap
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
