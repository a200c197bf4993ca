"""Plain FP64 products at the edges of the fragment kernel's tiles and splits.

Rows and columns around multiples of 16, 32 and 64 (each tile shape and its last,
partly empty tile), contractions around multiples of 4 and 8 (the masked steps),
shorter than one step per wave, and long enough to be split.
"""
import numpy as np
import pytest
import torch

from paper_2407_18947_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 1), (5, 7, 3), (16, 16, 8), (17, 15, 9), (33, 65, 37), (3, 700, 12), (700, 3, 13),
    (64, 4100, 68), (4100, 64, 69), (260, 520, 262), (25, 324, 324), (48, 48, 2055), (1030, 1030, 5),
])
def test_products_at_tile_edges(M, N, K):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g = np.random.default_rng(M * 7919 + N * 31 + K)
    A = g.standard_normal((M, K)) + 1j * g.standard_normal((M, K))
    B = g.standard_normal((K, N)) + 1j * g.standard_normal((K, N))
    C = _lib.rtcc3_zgemm_selftest(A, B, 0)
    # each of K terms passes at most K roundings of sums of at most twice its
    # size (three real products per complex one), in any order of summation
    bound = 8 * (K + 8) * np.finfo(float).eps * (np.abs(A) @ np.abs(B))
    assert np.all(np.abs(C - A @ B) <= bound)
