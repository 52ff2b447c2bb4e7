"""Activations far below the largest one of their 32 (massive activations in single channels), two to sixteen rows: columns
whose weights are zero at the large ones are as exact as without them."""
import numpy as np
import pytest
import torch

from oracle import hlq_oracle as O
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth

from gpu_util import dev, pack_on_gpu

pytestmark = pytest.mark.gpu


WEIGHT = np.array([0.5, 0.25, 0.125, 0.125])[np.arange(32) // 2 % 4]   # of an activation by its place in the 32


def left_over(X):
    """Bound on what the terms leave of every activation: 2^-20 of the largest of its 32 by four terms, as weighted; 2^-36 in
    eight, which a block has where all eight of a place are 2^-8 of the largest (or less), as weighted, and not all zero."""
    w = np.abs(X.astype(np.float64)).reshape(X.shape[0], -1, 32) * WEIGHT
    most = np.stack([w[..., np.arange(32) // 2 % 4 == r].max(-1) for r in range(4)], -1)
    exponent = np.maximum(np.floor(np.log2(np.maximum(most / WEIGHT[::2][:4], 2.0 ** -24))), -14) + np.log2(WEIGHT[::2][:4])
    wide = exponent.max(-1) - np.where(most > 0, exponent, 99).min(-1) > 8
    left = np.where(wide, 2.0 ** -36, 2.0 ** -20)[..., None] * w.max(-1, keepdims=True) / WEIGHT
    return left.reshape(X.shape), wide


def check(K, N, q, G, M, ratio, share, key):
    """One channel of a share of the 32-blocks (of one at least) is `ratio` times the others; codes and zeros are zero there.  The sums are fp32
    over the planes one by one (2^-20 of the sum of the magnitudes that are added is ample for K <= 8192)."""
    codes, S, Z = synth.make_weight(K, N, q, G, "wide", key)
    Z[:] = 0
    rng = np.random.default_rng(K + N + M + int(ratio))
    large = 32 * np.flatnonzero((rng.random(K // 32) < share) | (np.arange(K // 32) == K // 50))
    large = large + rng.integers(0, 32, large.size)
    codes[large] = 0
    X = synth.make_x(M, K, "wide", key)
    X[:, large] = (ratio * rng.uniform(1.0, 2.0, (M, large.size)) * np.where(rng.random((M, large.size)) < 0.5, -1, 1)).astype(np.float16)
    left, wide = left_over(X)
    assert ratio < 8000 or wide.any()
    desc, packed = pack_on_gpu(codes, S, Z, q, G)
    ws = B.alloc_workspace(desc, M)
    Y = torch.empty((M, N), dtype=torch.float32, device="cuda")
    for _ in range(2):
        B.hlq_lut_gemm(desc, packed, dev(X), Y, out_f32=True, ws=ws)
    planes = np.repeat(S.astype(np.float64).sum(0), G, 0)
    x = np.abs(X.astype(np.float64))
    x[:, large] = 0
    assert (np.abs(Y.cpu().numpy().astype(np.float64) - O.gemm_dequant(X, codes, S, Z, q, G)) <= (2.0 ** -20 * x + left) @ planes).all()


@pytest.mark.parametrize("ratio", [100.0, 8000.0, 32000.0])
@pytest.mark.parametrize("M", [3, 4, 7, 8, 16])
@pytest.mark.parametrize("q,G", [(2, 128), (4, 128), (3, 256)])
def test_many_rows_kernel(q, G, M, ratio):
    B.set_gemm_path(B.GEMM_ROWS16)
    try:
        check(1152 if G == 128 else 1280, 136, q, G, M, ratio, 0.3, "rows")
        check(4096, 72, q, G, M, ratio, 1.0, "rows")
    finally:
        B.set_gemm_path(B.GEMM_AUTO)


# one step a wavefront, several windows of one column block, several column blocks of one window, both; a narrow last tile
@pytest.mark.parametrize("K,N,G", [(4096, 1032, 128), (8192, 3208, 64), (2048, 2056, 32), (2304, 4104, 128), (4096, 5400, 128), (8192, 4040, 256)])
@pytest.mark.parametrize("M", [2, 3, 4])
@pytest.mark.parametrize("ratio,share", [(1000.0, 1.0), (8000.0, 0.03), (32000.0, 0.3)])
def test_few_rows_kernel(K, N, G, M, ratio, share):
    check(K, N, 2, G, M, ratio, share, "few")
