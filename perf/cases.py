"""The workloads this library is measured on, one dict each, and how to run them.

A data-parallel step compresses every worker's gradient (encode), sums the
sketches and ORs the indexes (aggregate) and recovers the exact sum (decode).
A worker's process calls the encode and the decode; a single process that
simulates all workers calls all three.  The cases take both forms, over the
gradient shapes of the configured models (embedding table, LSTM, VGG19,
BERT-base), from 2^16 to 2^30 parameters, for both value types, both sketch
layouts, both index kinds and every input and output form of the calls.

A case's fields:
  op        "iteration" (W encodes, aggregate, decode), "encode" (one
            worker), "decode" (of a given aggregate), "roundtrip" (one
            worker's encode and the decode of its own sketch)
  n         gradient length
  vtype     "i32" (fixed point at scale 2^20) or "f32"
  sketch    "global" or "blocked"
  index     "bitmap" or "bloom"
  encode    "atomic" (hc_encode), "staged" (hc_encode_staged), "gather"
            (hc_encode_gather), "coo" (hc_encode_coo); absent for "decode"
  support   "spread" (uniform positions) or "rows" (whole rows of `dim`
            consecutive parameters, row ids drawn by Zipf(1.1) rank)
  workers, density, overlap   (spread) every worker has density * n nonzeros,
            the fraction `overlap` of them shared by all workers and the
            others its own; for "decode" the aggregate has density * n
  dim, touched                (rows) the row length and the number of rows
  gamma     sketch cells per aggregate nonzero
  out       "dense" (dense sum and recovered mask), "coo" (index and value
            list) or "both"
  plan      whether the decode has the geometry's inverse row map
"""
import math

import numpy as np
import torch

import paper_2402_07529_amd as hc

HASH_SEED = 2024
SCALE = 2.0**20


def _case(name=None, **kw):
    base = dict(op="decode", n=0, vtype="i32", sketch="global", index="bitmap", encode="atomic",
                support="spread", workers=1, density=0.01, overlap=0.0, dim=64, touched=0,
                gamma=1.23, out="dense", plan=True)
    base.update(kw)
    if name is not None:
        base["name"] = name
    return base


def listed():
    return [
        # the smallest step: a 2^16-parameter model on four workers, where only
        # launches and round trips count
        _case("small_step_i32", op="iteration", n=65536, workers=4, density=655 / 65536, overlap=0.5),
        # a small ragged fp32 model on eight workers, dense and list outputs
        _case("ragged_step_f32", op="iteration", n=1500007, vtype="f32", encode="staged", workers=8,
              density=0.02, overlap=0.5, gamma=1.3, out="both"),
        # one worker's gradient of a 2^24 x 64 embedding table: 4096 rows touched
        _case("embedding_encode_i32", op="encode", n=2**30, support="rows", touched=4096),
        # the sum over eight such workers (24,245 distinct rows) recovered
        _case("embedding_decode_i32", n=2**30, support="rows", touched=24245),
        # one worker's VGG19 gradient at 1 % density
        _case("vgg19_encode_i32", op="encode", n=143667240, encode="staged", density=0.01,
              gamma=1.23 * 5.9),
        # the sum of eight workers' VGG19 gradients (30 % overlap: 5.9 % dense)
        _case("vgg19_decode_i32", n=143667240, density=0.059),
        # the same for the LSTM in fp32, whose length is 2 mod 4
        _case("lstm_decode_f32", n=85974278, vtype="f32", density=0.059),
        # a whole simulated step of sixteen BERT-base workers, blocked sketch
        _case("bert_blocked_step_i32", op="iteration", n=109482240, sketch="blocked", workers=16,
              density=0.01, overlap=0.5, gamma=1.3, plan=False),
        # recovery of the VGG19 sum from a blocked fp32 sketch
        _case("vgg19_blocked_decode_f32", n=143667240, vtype="f32", sketch="blocked", density=0.059,
              gamma=1.3, plan=False),
        # one worker, the natural density of an unsparsified VGG19 gradient,
        # the sketch as long as the gradient: compress and decompress
        _case("vgg19_natural_roundtrip_i32", op="roundtrip", n=143667240, encode="gather",
              density=0.696, gamma=1 / 0.696),
        # sixteen sparse BERT-base workers with a Bloom-filter index
        _case("bert_bloom_step_i32", op="iteration", n=109482240, index="bloom", workers=16,
              density=0.001, overlap=0.9),
        # one worker whose sparsifier hands over (index, value) pairs
        _case("bert_coo_encode_f32", op="encode", n=109482240, vtype="f32", encode="coo",
              density=0.01, gamma=1.23 * 8.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    vtype = rng.choice(["i32", "i32", "f32"])
    kind = rng.choice(["iteration", "iteration", "encode", "encode", "decode", "decode", "decode",
                       "embedding", "natural"])
    density = math.exp(rng.uniform(math.log(0.0005), math.log(0.03)))
    gamma = 1.4 if vtype == "f32" else rng.choice([1.23, 1.3, 1.5])
    out = rng.choice(["dense", "dense", "both", "coo"])
    if kind == "embedding":
        dim = rng.choice([16, 64, 128])
        rows = _log(rng, 2**13, 2**30 // dim)
        op = rng.choice(["encode", "decode"])
        touched = max(16, min(rows // 16, _log(rng, 64, 24000)))
        return _case(op=op, n=rows * dim, vtype=vtype, support="rows", dim=dim, touched=touched,
                     gamma=gamma, out=out)
    if kind == "natural":
        return _case(op="roundtrip", n=_log(rng, 70000, 30_000_000), vtype=vtype, encode="gather",
                     density=rng.uniform(0.3, 0.75), gamma=1.5, out="dense")
    if kind == "iteration":
        workers = rng.choice([2, 4, 8])
        overlap = rng.choice([0.1, 0.5, 0.9])
        n = _log(rng, 65536, 30_000_000)
        sketch = "blocked" if n > 2_000_000 and rng.random() < 0.5 else "global"
        index = "bloom" if sketch == "global" and rng.random() < 0.3 else "bitmap"
        encode = rng.choice(["atomic", "staged"]) if sketch == "global" else "atomic"
        return _case(op="iteration", n=n, vtype=vtype, sketch=sketch, index=index, encode=encode,
                     workers=workers, density=density, overlap=overlap,
                     gamma=max(gamma, 1.4) if sketch == "blocked" else gamma, out=out,
                     plan=sketch == "global" and rng.random() < 0.8)
    n = _log(rng, 65536, 140_000_000)
    if kind == "encode":
        encode = rng.choice(["atomic", "staged", "coo", "blocked"])
        if encode == "blocked":
            return _case(op="encode", n=max(n, 2_000_000), vtype=vtype, sketch="blocked",
                         density=density, gamma=1.4)
        return _case(op="encode", n=n, vtype=vtype, encode=encode, density=density, gamma=1.23 * 6)
    sketch = "blocked" if n > 2_000_000 and rng.random() < 0.4 else "global"
    return _case(op="decode", n=n, vtype=vtype, sketch=sketch, density=min(0.1, 4 * density),
                 gamma=max(gamma, 1.4) if sketch == "blocked" else gamma, out=out,
                 plan=sketch == "global" and rng.random() < 0.8)


# ---- sizes that follow from a case alone ------------------------------------------

def _counts(case):
    """(nonzeros of one worker, of them shared by all, nonzeros of the union)."""
    if case["support"] == "rows":
        m = case["touched"] * case["dim"]
        return m, 0, m
    m = max(1, int(round(case["density"] * case["n"])))
    s = int(round(case["overlap"] * m))
    return m, s, s + case["workers"] * (m - s)


def _params(case):
    union = _counts(case)[2]
    if case["sketch"] == "blocked":
        return hc.hc_geometry_blocked(case["n"], union, case["gamma"], 1024, 0, HASH_SEED,
                                      case["vtype"])
    if case["index"] == "bloom":
        return hc.hc_geometry_bloom(case["n"], union, case["gamma"], 1024, HASH_SEED,
                                    case["vtype"])[0]
    return hc.hc_geometry(case["n"], union, case["gamma"], 1024, HASH_SEED, case["vtype"])


def _max_support(case, p):
    union = _counts(case)[2]
    if case["index"] == "bloom":  # room for the filter's false positives
        return int(union + 4 * 2.0 ** -int(p.bloom_k) * (case["n"] - union)) + 1024
    return union


# ---- inputs ------------------------------------------------------------------------

def _distinct(n, m, gen):
    """m distinct positions below n, in random order."""
    if 2 * m > n or n < 4096:
        return torch.randperm(n, device="cuda", generator=gen)[:m]
    got = torch.empty(0, dtype=torch.int64, device="cuda")
    while got.numel() < m:
        need = int((m - got.numel()) * (1.1 + m / n)) + 64
        more = torch.randint(0, n, (need,), device="cuda", generator=gen)
        got = torch.unique(torch.cat([got, more]))
    return got[torch.randperm(got.numel(), device="cuda", generator=gen)[:m]]


def _values(count, case, gen):
    """Gradient values N(0, 10^-3) (embedding rows: 10^-2), none zero."""
    v = torch.randn(count, device="cuda", generator=gen) * (1e-2 if case["support"] == "rows" else 1e-3)
    if case["vtype"] == "f32":
        return torch.where(v == 0, torch.full_like(v, 1e-4), v)
    q = torch.round(v * SCALE).to(torch.int32)
    return torch.where(q == 0, torch.ones_like(q), q)


def _zipf_rows(rows, count, seed):
    """count distinct row ids: Zipf(1.1) ranks through a random odd-multiplier map."""
    rng = np.random.default_rng(seed)
    kept = np.empty(0, np.int64)
    while True:
        r = rng.zipf(1.1, 4 * count)
        kept = np.concatenate([kept, r[r <= rows].astype(np.int64)])
        _, first = np.unique(kept, return_index=True)
        if first.size >= count:
            ranks = kept[np.sort(first)[:count]] - 1
            break
        if kept.size > 400 * count:  # a small table: the ranks left over, in order
            seen = kept[np.sort(first)] - 1
            rest = np.setdiff1d(np.arange(rows), seen, assume_unique=True)
            ranks = np.concatenate([seen, rest])[:count]
            break
    mult = int(rng.integers(0, rows)) * 2 + 1
    while math.gcd(mult, rows) != 1:
        mult += 2
    return (ranks * mult + int(rng.integers(0, rows))) % rows


def _gradients(case, seed):
    """Per worker: (positions ascending, values).  Lazily, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 13)
    n = case["n"]
    if case["support"] == "rows":
        rows = torch.from_numpy(_zipf_rows(n // case["dim"], case["touched"], seed)).cuda()
        rows = torch.sort(rows).values
        idx = (rows[:, None] * case["dim"] + torch.arange(case["dim"], device="cuda")).reshape(-1)
        yield idx, _values(idx.numel(), case, gen)
        return
    m, s, union = _counts(case)
    pos = _distinct(n, union, gen)
    for w in range(case["workers"]):
        own = pos[s + w * (m - s):s + (w + 1) * (m - s)]
        idx = torch.sort(torch.cat([pos[:s], own])).values
        yield idx, _values(m, case, gen)


def _dense(case, idx, val, dtype=None):
    x = torch.zeros(case["n"], dtype=val.dtype if dtype is None else dtype, device="cuda")
    x[idx] = val if dtype is None else val.to(dtype)
    return x


def _encode(st, w, y, b):
    p, how = st["p"], st["encode"]
    if how == "coo":
        hc.hc_encode_coo(p, st["idx"][w], st["val"][w], y, b)
    elif how == "staged":
        hc.hc_encode_staged(p, st["plan"], st["stage"], st["x"][w], y, b)
    elif how == "gather":
        hc.hc_encode_gather(p, st["plan"], st["x"][w], y, b)
    else:
        hc.hc_encode(p, st["x"][w], y, b)


def prepare(case, seed):
    """The gradients (or, for a decode, the aggregated sketch and index), the
    geometry, its plan where the calls take one, workspaces and outputs."""
    p = _params(case)
    vt = torch.float32 if case["vtype"] == "f32" else torch.int32
    W, op, n = case["workers"], case["op"], case["n"]
    st = dict(op=op, p=p, W=W, encode=case["encode"])
    needs_plan = case["plan"] and case["sketch"] == "global" and op != "encode"
    if needs_plan or case["encode"] in ("staged", "gather"):
        st["plan"] = hc.make_plan(p)
    st["decode_plan"] = st.get("plan") if needs_plan else None
    if case["encode"] == "staged":
        st["stage"] = hc.alloc_stage_workspace(p)

    def empty(*shape, dtype=vt):
        return torch.empty(shape, dtype=dtype, device="cuda")

    st["y"], st["b"] = empty(p.cells), empty(p.index_words, dtype=torch.int32)
    if op == "decode":
        # the aggregate arrives from the network; here it is the sketch of the sum
        idx, val = next(_gradients(case, seed))
        hc.hc_encode_coo(p, idx.to(torch.int32), val, st["y"], st["b"])
    elif case["encode"] == "coo":
        pairs = list(_gradients(case, seed))
        st["idx"] = [i.to(torch.int32) for i, _ in pairs]
        st["val"] = [v for _, v in pairs]
    else:
        st["x"] = [_dense(case, i, v) for i, v in _gradients(case, seed)]
    if op == "iteration":
        st["yw"], st["bw"] = empty(W, p.cells), empty(W, p.index_words, dtype=torch.int32)
    if op != "encode":
        cap = _max_support(case, p)
        st["cap"] = cap
        st["ws"] = hc.alloc_workspace(p, cap)
        st["info"] = hc.alloc_info()
        st["out"] = {}
        if case["out"] in ("dense", "both"):
            st["out"]["x_out"] = empty(n)
            st["out"]["mask"] = empty(p.words, dtype=torch.int32)
        if case["out"] in ("coo", "both"):
            # entries past the support are not written
            size = cap
            st["out"]["coo_idx"] = torch.zeros(size, dtype=torch.int32, device="cuda")
            st["out"]["coo_val"] = torch.zeros(size, dtype=vt, device="cuda")
    return st


def run(st):
    p, op = st["p"], st["op"]
    y, b = st["y"], st["b"]
    if op == "iteration":
        for w in range(st["W"]):
            _encode(st, w, st["yw"][w], st["bw"][w])
        hc.hc_aggregate(p, st["yw"], st["bw"], st["W"], y, b)
    elif op != "decode":
        _encode(st, 0, y, b)
    got = {} if op == "decode" else {"y": y, "b": b}
    if op != "encode":
        hc.hc_decode(p, y, b, st["info"], st["ws"], max_support=st["cap"], plan=st["decode_plan"],
                     **st["out"])
        got.update(st["out"])
        got["info"] = st["info"][:hc.INFO_BYTES]
    return got


# ---- what a pass cannot do without -------------------------------------------------

def work(case):
    p = _params(case)
    n, W, (m, _, union) = case["n"], case["workers"], _counts(case)
    sketch = 4 * p.cells + 4 * p.index_words
    nbytes = adds = 0
    if case["op"] != "decode":
        nbytes += 8 * m if case["encode"] == "coo" else 4 * n * W  # the gradients
        nbytes += sketch                                           # the (summed) sketch and index
        adds += 3 * m * W
    else:
        nbytes += sketch                                           # the aggregate, read
    if case["op"] == "iteration":
        adds += (W - 1) * p.cells
    if case["op"] != "encode":
        if case["out"] in ("dense", "both"):
            nbytes += 4 * n + 4 * p.words
        if case["out"] in ("coo", "both"):
            nbytes += 8 * union
        adds += 3 * union
    return {"bytes": nbytes, "flops": adds}


# ---- correctness -------------------------------------------------------------------

def tolerance(case):
    # int32 sums wrap and peel exactly: every output is the same whatever the
    # order.  fp32: sketches are summed in fp32 by atomics in no fixed order, and
    # the peel carries a cell's rounding along chains of subtractions.  Two runs
    # on the same inputs differed by up to 8.1e-7 (2-norm) and 5.7e-5 (largest)
    # in the recovered sum of 5 M nonzeros, and by 8e-8 in smaller ones and in
    # the sketches; this is four times that.
    return "exact" if case["vtype"] == "i32" else {"rel": 3.2e-6, "max": 2.3e-4}


_M64 = (1 << 64) - 1


def _i64(v):
    v &= _M64
    return v - (1 << 64) if v >> 63 else v


def _shr(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _splitmix(i):
    """SplitMix64 output number i (an int64 tensor) of HASH_SEED."""
    z = (i + 1) * _i64(0x9E3779B97F4A7C15) + HASH_SEED
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _plain_sketch(p, idx, val):
    """The Count Sketch of (idx, val) in 64 bits, global or blocked."""
    c, K = int(p.c), int(p.block)
    rows = int(p.block_rows) if K else int(p.rows)  # the rows a batch draws from
    batch, t = idx // c, idx % c
    h = [_splitmix(3 * batch + j) for j in range(3)]
    lo = [v & 0xFFFFFFFF for v in h]
    r0 = (lo[0] * rows) >> 32
    r1 = (lo[1] * (rows - 1)) >> 32
    r1 = r1 + (r1 >= r0)
    a, b = torch.minimum(r0, r1), torch.maximum(r0, r1)
    r2 = (lo[2] * (rows - 2)) >> 32
    r2 = r2 + (r2 >= a)
    r2 = r2 + (r2 >= b)
    r = [r0, r1, r2]
    bias = [_shr(v, 32) % c for v in h]
    if K:
        # rows ascending within the block; the rotations offset from the first
        # by the digits of a keyed bijection of the batch's number in the block
        r = [torch.minimum(a, r2), r0 + r1 + r2 - torch.minimum(a, r2) - torch.maximum(b, r2),
             torch.maximum(b, r2)]
        q = batch // K
        u, M = _splitmix(q + (1 << 62)), c * c
        half = c.bit_length() - 1
        x = (batch - q * K + (_shr(u, 40) & 0xFFFFF)) % M
        x = (x * ((u & 0xFFFFF) | 1)) % M
        x = x ^ (x >> half)
        x = (x * ((_shr(u, 20) & 0xFFFFF) | 1)) % M
        x = x ^ (x >> half)
        bias[1], bias[2] = (bias[0] + x % c) % c, (bias[0] + x // c) % c
        r = [v + q * rows for v in r]
    y = torch.zeros(p.cells, dtype=val.dtype, device="cuda")
    for j in range(3):
        y.index_add_(0, r[j] * c + (t + bias[j]) % c, torch.where(h[j] < 0, -val, val))
    return y


def exact(case, seed):
    """The sum of the gradients and its sketch in 64 bits (the decode recovers
    the exact sum; its mask, index and summary are whole numbers)."""
    p = _params(case)
    f32 = case["vtype"] == "f32"
    wide = torch.float64 if f32 else torch.int64
    total = torch.zeros(case["n"], dtype=wide, device="cuda")
    member = torch.zeros(case["n"], dtype=torch.bool, device="cuda")
    for idx, val in _gradients(case, seed):
        total[idx] += val.to(wide)
        member[idx] = True
    idx = torch.nonzero(member).reshape(-1)
    val = total[idx]
    got = {}
    if case["op"] != "decode":
        got["y"] = _plain_sketch(p, idx, val)
        got["b"] = None
    if case["op"] != "encode":
        if case["out"] in ("dense", "both"):
            got["x_out"], got["mask"] = total, None
        if case["out"] in ("coo", "both"):
            # a Bloom filter's list holds its false positives (value 0) too
            bitmap = case["index"] == "bitmap"
            got["coo_idx"], got["coo_val"] = (idx, val) if bitmap else (None, None)
        got["info"] = None
    return got
