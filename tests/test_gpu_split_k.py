"""GPU: the split-K GEMM where its requests meet an edge: a last chunk of half size, a second chunk of a pair that is missing or
half there, weight tiles that end inside a work-group."""
import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si
from oracle import stairs_oracle as so

pytestmark = pytest.mark.gpu


# 9..16 rows take two 512-wide chunks per work-group, the others one; 1, 5 and 17 tiles: a wave without a tile of its own
@pytest.mark.parametrize("K", [256, 512, 1280, 1536, 1792, 16640])
@pytest.mark.parametrize("N", [16, 80, 272])
def test_edges_of_chunks_and_tiles(N, K):
    print(f"split-K N={N} K={K}", flush=True)
    rng = np.random.default_rng([N, K])
    W = si.bf16_round(rng.standard_normal((N, K), dtype=np.float32))
    X = rng.standard_normal((32, K), dtype=np.float32)
    Wr = so._decode(W, np.float64)
    ref = X.astype(np.float64) @ Wr.T
    # x as bf16 high + low parts is exact to 2^-16 of its size, fp32 sums of K products to K 2^-24 of the sum of sizes
    bound = (2.0 ** -16 + K * 2.0 ** -24) * (np.abs(X).astype(np.float64) @ np.abs(Wr).T)
    wide = pkg.stairs_gemm_host(W, X)
    assert np.all(np.abs(wide - ref) <= bound)
    for m in (5, 8, 9, 15, 16, 17):
        assert np.array_equal(pkg.stairs_gemm_host(W, X[:m]), wide[:m]), m
