"""Two to four rows on the one-row kernel (hlq_gemv_cols.hip): every format, a row more than the call has, ragged tiles, odd chunk
counts, one step and several, K slices, strided rows, magnitudes far apart, infinities and NaNs."""
import numpy as np
import pytest
import torch

from oracle import hlq_oracle as O
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth

from gpu_util import dev, pack_on_gpu

pytestmark = pytest.mark.gpu


def on_the_one_row_kernel(K, N, q, G, M):
    """Whether the launch is planned for it: wavefronts by windows of four chunks, and workgroups that do not own whole tiles."""
    info = B.gemv_plan_query([B.make_desc(K, N, q, G)], M)[0]
    kw = 1
    while kw * 2 <= 8 and kw < -(-K // 512):
        kw *= 2
    return info.waves_per_workgroup == 8 and info.waves_per_tile == kw and info.tile_groups != -(-(-(-N // 64)) // (8 // kw))


def product(K, N, q, G, X, pad=0, key="few", cols=slice(None)):
    """fp32 result, reference, and a bound: what the terms leave of an activation is at most 2^-18 of the largest of its word
    (32 k), the sums are fp32 over the planes one by one (2^-20 of the sum of magnitudes is ample for K <= 8192)."""
    codes, S, Z = synth.make_weight(K, N, q, G, "few", key)
    M = X.shape[0]
    desc, packed = pack_on_gpu(codes, S, Z, q, G)
    xbuf = torch.full((M, K + 8 * pad), float("nan"), dtype=torch.float16, device="cuda")
    xbuf[:, :K] = dev(X)
    ybuf = torch.full((M, N + 3 * pad), 7.0, dtype=torch.float32, device="cuda")
    ws = B.alloc_workspace(desc, M)
    for _ in range(2):   # the second call finds the workspace as the first one left it
        B.hlq_lut_gemm(desc, packed, xbuf[:, :K], ybuf[:, :N], out_f32=True, ws=ws)
    Y = ybuf.cpu().numpy().astype(np.float64)
    assert (Y[:, N:] == 7.0).all() and int(ws[:131072].view(torch.int32).abs().sum()) == 0
    x = np.abs(X.astype(np.float64))
    codes, S, Z = codes[:, cols], S[:, :, cols], Z[:, cols]
    planes = np.repeat(S.astype(np.float64).sum(0) + np.abs(Z.astype(np.float64)), G, 0)
    largest = np.repeat(x.reshape(M, K // 32, 32).max(2), 32, 1)
    return Y[:, :N][:, cols], O.gemm_dequant(X, codes, S, Z, q, G), 2.0 ** -18 * largest @ planes + 2.0 ** -20 * x @ planes


@pytest.mark.parametrize("M", [2, 3, 4])
@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("G", [32, 64, 128, 256])
def test_formats(q, G, M):
    K = 2304 if G < 256 else 2560          # 18 or 20 chunks: five windows, the last one short
    assert on_the_one_row_kernel(K, 1096, q, G, M)
    Y, ref, bound = product(K, 1096, q, G, synth.make_x(M, K, "few", outliers=True), pad=1)
    assert (np.abs(Y - ref) <= bound).all()


@pytest.mark.parametrize("K,N", [(8192, 3208), (8064, 3400), (1536, 8200), (4096, 520), (4096, 4096), (2048, 12168)])
def test_one_step_and_several(K, N):
    for M in (2, 4):
        assert on_the_one_row_kernel(K, N, 2, 128, M)
        Y, ref, bound = product(K, N, 2, 128, synth.make_x(M, K, "few"))
        assert (np.abs(Y - ref) <= bound).all()


# a wavefront walks over several column blocks, within a tile, into the next one and into a narrow last one: the largest launches of
# up to 4096 chunk-tiles, and the smallest from 14000 or 18000 on (groups of 32 and 64).  Results of the first and last tiles and some between
@pytest.mark.parametrize("K,N,q,G,M", [(4096, 8136, 2, 128, 4), (4096, 8072, 4, 256, 3), (2048, 16328, 1, 64, 4), (1024, 112072, 2, 64, 4), (1024, 144072, 4, 64, 3),
                                       (1024, 144072, 2, 32, 2), (128, 896136, 1, 32, 3), (8192, 14216, 3, 32, 4)])
def test_several_column_blocks(K, N, q, G, M):
    info = B.gemv_plan_query([B.make_desc(K, N, q, G)], M)[0]
    assert on_the_one_row_kernel(K, N, q, G, M)
    assert info.tile_groups * (info.waves_per_workgroup // info.waves_per_tile) < -(-N // 16)
    cols = np.unique(np.concatenate([np.arange(0, 200), np.arange(N - 200, N), np.random.default_rng(N).integers(0, N, 400)]))
    Y, ref, bound = product(K, N, q, G, synth.make_x(M, K, "few"), cols=cols)
    assert (np.abs(Y - ref) <= bound).all()


@pytest.mark.parametrize("W,cpw", [(8, 1), (4, 2), (2, 3)])
def test_slices(W, cpw):
    B.set_gemv_plan(0, W, cpw)
    try:
        for M in (2, 3):
            Y, ref, bound = product(4096, 776, 3, 64, synth.make_x(M, 4096, "few"))
            assert (np.abs(Y - ref) <= bound).all()
    finally:
        B.set_gemv_plan(0, 0, 0)


@pytest.mark.parametrize("spread", [12, 30])
def test_magnitudes_far_apart_inside_a_word(spread):
    K, M = 2048, 4
    rng = np.random.default_rng(spread)
    X = (np.exp2(rng.integers(-spread, 1, size=(M, K)).astype(np.float64)) * rng.uniform(-2.0, 2.0, size=(M, K)) * 2.0 ** 14).astype(np.float16)
    Y, ref, bound = product(K, 1032, 2, 128, X)
    assert (np.abs(Y - ref) <= bound).all()


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_row_with_an_infinity_or_nan(bad):
    """is NaN as a whole; the other rows are what they are without it."""
    K, M = 2048, 3
    X = synth.make_x(M, K, "few-nan")
    clean, _, _ = product(K, 1032, 3, 128, X)
    X[1, 777] = bad
    Y, _, _ = product(K, 1032, 3, 128, X)
    assert np.isnan(Y[1]).all() and np.array_equal(Y[[0, 2]], clean[[0, 2]])
