"""The many-rows kernel's activation terms: blocks of 32 activations share a power of two, four terms each."""
import numpy as np
import pytest
import torch

from oracle import hlq_oracle as O
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth
from gpu_util import dev, pack_on_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def many_rows_kernel():
    B.set_gemm_path(B.GEMM_ROWS16)
    yield
    B.set_gemm_path(B.GEMM_AUTO)


@pytest.mark.parametrize("M", [3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("spread", [0, 12, 30])
def test_magnitudes_far_apart_inside_a_block(M, spread):
    """What the terms leave of an activation is at most 2^-20 of its block's largest as weighted by the plane codes (1/2 to
    1/8), 2^-18 as it is; the sums are fp32 (2^-20 of the sum of magnitudes is ample for K = 384)."""
    K, N, q, G = 384, 72, 2, 128
    codes, S, Z = synth.make_weight(K, N, q, G, "rows-terms")
    rng = np.random.default_rng(M * 100 + spread)
    mag = np.exp2(rng.integers(-spread, 1, size=(M, K)).astype(np.float64)) * rng.uniform(1.0, 2.0, size=(M, K))
    X = (np.where(rng.random((M, K)) < 0.5, -1.0, 1.0) * mag * 2.0 ** 14).astype(np.float16)
    desc, packed = pack_on_gpu(codes, S, Z, q, G)
    Y = B.hlq_lut_gemm(desc, packed, dev(X), out_f32=True).cpu().numpy().astype(np.float64)
    ref = O.gemm_dequant(X, codes, S, Z, q, G)
    planes = np.repeat(S.astype(np.float64).sum(0) + np.abs(Z.astype(np.float64)), G, 0)   # the planes are added one by one
    largest = np.repeat(np.abs(X.astype(np.float64)).reshape(M, K // 32, 32).max(2), 32, 1)
    bound = 2.0 ** -18 * largest @ planes + 2.0 ** -20 * np.abs(X.astype(np.float64)) @ planes
    assert (np.abs(Y - ref) <= bound).all()


@pytest.mark.parametrize("M", [4, 7, 16])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_row_with_an_infinity_or_nan(M, bad):
    """is NaN as a whole; the other rows are what they are without it."""
    K, N, q, G = 256, 64, 3, 128
    codes, S, Z = synth.make_weight(K, N, q, G, "rows-nan")
    X = synth.make_x(M, K, "rows-nan")
    desc, packed = pack_on_gpu(codes, S, Z, q, G)
    clean = B.hlq_lut_gemm(desc, packed, dev(X), out_f32=True).cpu()
    X[M - 2, 131] = bad
    Y = B.hlq_lut_gemm(desc, packed, dev(X), out_f32=True).cpu()
    others = [m for m in range(M) if m != M - 2]
    assert torch.isnan(Y[M - 2]).all() and torch.equal(Y[others], clean[others])
