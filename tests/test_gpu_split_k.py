"""GPU: the split-K GEMM where its requests meet an edge: a last chunk of half size, a second chunk of a pair that is missing or
half there, weight tiles that end inside a work-group, one and two tiles per wave, every number of rows that has a form of its own."""
import ctypes as C

import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si
from oracle import stairs_oracle as so

pytestmark = pytest.mark.gpu

HEAD = 4                                               # the role stairs_gemm_host runs


class _WideCfg(C.Structure):
    _fields_ = [("nt", C.c_int), ("nw", C.c_int)]


def takes_split_k(m, N, K):
    lds = pkg.lib()._ZN6stairs13rows_path_ldsEiiii
    lds.restype, lds.argtypes = C.c_size_t, [C.c_int] * 4
    wide = pkg.lib()._ZN6stairs8wide_cfgEiiii
    wide.restype, wide.argtypes = _WideCfg, [C.c_int] * 4
    return lds(HEAD, m, N, K) == 0 and (m <= 4 or wide(HEAD, m, N // 16, K).nt == 0)


def check(N, K, rows, m_first):
    """rows[0] rows against 64 bits, fewer rows against the bits of those; from m_first rows on all of them take the kernel"""
    rng = np.random.default_rng([N, K])
    W = np.empty((N, K), np.uint16)
    X = rng.standard_normal((rows[0], K), dtype=np.float32)
    ref, size = np.empty((rows[0], N)), np.empty((rows[0], N))
    for n in range(0, N, 512):                         # (long matrices: a piece of the reference at a time)
        W[n:n + 512] = si.bf16_round(rng.standard_normal((min(512, N - n), K), dtype=np.float32))
        Wr = so._decode(W[n:n + 512], np.float64)
        ref[:, n:n + 512] = X.astype(np.float64) @ Wr.T
        size[:, n:n + 512] = np.abs(X).astype(np.float64) @ np.abs(Wr).T
    # x as bf16 high + low parts is exact to 2^-16 of its size, fp32 sums of K products to K 2^-24 of the sum of sizes
    bound = (2.0 ** -16 + K * 2.0 ** -24) * size
    most = pkg.stairs_gemm_host(W, X)
    assert np.all(np.abs(most - ref) <= bound)
    for m in rows[1:]:
        assert np.array_equal(pkg.stairs_gemm_host(W, X[:m]), most[:m]), m
    assert [m for m in rows if takes_split_k(m, N, K)] == [m for m in rows if m >= m_first]


# 9..16 rows take two 512-wide chunks per work-group, the others one; 1, 5 and 17 tiles: a wave without a tile of its own.
# Chunks: 9 whole ones, 10 and 11 whose last is half there, 10 and 22 whole ones, 33 whose last is half there.  (Beyond 4096 only:
# shorter k is other kernels' work, held to the same bits in the test behind this one.)
@pytest.mark.parametrize("K,m_first", [(4608, 4), (4864, 4), (5120, 4), (5376, 4), (11008, 2), (16640, 2)])
@pytest.mark.parametrize("N", [16, 80, 272])
def test_edges_of_chunks_and_tiles(N, K, m_first):
    print(f"split-K N={N} K={K}", flush=True)
    check(N, K, (32, 17, 16, 15, 9, 8, 5, 4, 3, 2, 1), m_first)


@pytest.mark.parametrize("K", [256, 512, 1280, 1536, 1792])
@pytest.mark.parametrize("N", [16, 80, 272])
def test_shorter_k_on_the_other_kernels(N, K):
    print(f"N={N} K={K}", flush=True)
    check(N, K, (32, 17, 16, 15, 9, 8, 5), 33)


# Enough column groups for two tiles per wave: the request two units ahead is the next tile's, at a pair's end the next chunk's.
# 301 and 191 tiles: in the last work-group some waves have a second tile, others one; 1..16 rows, and 17..32 (which need few tiles).
@pytest.mark.parametrize("N,K,rows", [(4816, 16640, (16, 9, 8, 5, 4, 2)), (3056, 22272, (32, 17))])
def test_two_tiles_per_wave(N, K, rows):
    print(f"split-K N={N} K={K}", flush=True)
    check(N, K, rows, 1)
