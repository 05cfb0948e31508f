"""Bloom-filter inserts and probes by tile against the oracle: batches of 256,
512 and 1024 parameters with few and with many nonzero words, hash counts on
both sides of a half wave, and lengths whose last wave is partial.  Filters,
sketches and decodes are bit-exact."""
import numpy as np
import pytest

import workloads as wl
from hc_pipeline import gpu_run, oracle_run
from test_gpu_parity import assert_same_info

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [256, 512, 1024])
@pytest.mark.parametrize("n,density,k", [
    (1_200_003, 0.0008, 5),          # about one nonzero per batch of 1024
    (1_200_003, 0.004, 13),          # around the few-words bound
    (200 * 1024 + 33, 0.05, 33),     # most words nonzero, more hashes than half a wave
    (64 * 1024, 0.01, 64), (1025, 0.2, 31), (31, 0.4, 32),
])
def test_bloom_tiles(n, density, k, c):
    w = wl.make("synthetic", "i32", n=n, W=2, density=max(density, 1.5 / n), overlap=0.5,
                data_seed=k, hash_seed=c)
    rows = max(3, int(1.4 * max(w.n_agg, 1)) // c + 2)
    brows = max(1, int(k * w.n_agg / 0.69) // c + 1)
    g = gpu_run(w, rows, c, bloom_k=k, bloom_rows=brows, use_plan=True)
    o = oracle_run(w, rows, c, bloom_k=k, bloom_rows=brows)
    for i in range(w.W):
        assert np.array_equal(g["B"][i], o["B"][i])
        assert np.array_equal(g["Y"][i], o["Y"][i])
    assert np.array_equal(g["x"], o["x"])
    assert np.array_equal(g["mask"], o["mask"])
    assert_same_info(g["info"], o["info"])
