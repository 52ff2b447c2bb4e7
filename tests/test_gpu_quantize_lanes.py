"""hlq_quantize with one, two and four lanes a group (chosen by the size of the launch): columns of launches of each kind
against the oracle, which treats columns one by one."""
import numpy as np
import pytest

from oracle import hlq_quantize_oracle as QO
from paper_2510_19482_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


# wavefronts of a launch with one lane a group: K / G x ceil(N / 64)
@pytest.mark.parametrize("K,N,G", [(2048, 2056, 64), (512, 2056, 64),                       # 1056: one, 264: two lanes
                                   (2048, 8200, 128), (2048, 1544, 128), (2048, 520, 128),  # 2064, 400, 144: one, two, four
                                   (4096, 2056, 256), (2048, 264, 256)])                    # 528, 40: two, four
@pytest.mark.parametrize("q", [1, 2, 3, 4])
def test_columns(K, N, G, q):
    rng = np.random.default_rng(K + N + G + q)
    W = (rng.standard_normal((K, N)) * 0.02).astype(np.float32)
    W[:, 1] = 0.013                                                          # equal weights
    W[:, 2] = (rng.integers(-1, 2, K) * 0.03).astype(np.float32)             # candidates coincide: its wavefront scans
    W[:, 3] = W[:, 3].view(np.uint32).__and__(0xffff0000).view(np.float32)   # 16-bit weights
    codes, S, Z, err = B.hlq_quantize(B.make_desc(K, N, q, G), dev(W), 4, with_err=True)
    cols = np.unique(np.concatenate([[0, 1, 3, 4, 63, 64, N - 1, N - 8], rng.integers(4, N, 12)]))
    ref, S_ref, Z_ref = QO.quantize(W[:, cols].astype(np.float64), q, G, t_max=4)
    assert np.array_equal(codes.cpu().numpy()[:, cols], ref)
    # fp16 parameters: one unit in the last place (2^-10 of the value) and the subnormals' spacing
    for got, want in ((S.cpu().numpy()[:, :, cols], S_ref), (Z.cpu().numpy()[:, cols], Z_ref)):
        assert (np.abs(got.astype(np.float64) - want) <= 2.0 ** -10 * np.abs(want) + 2.0 ** -24).all()
    err_ref = ((QO.reconstruct(ref, S_ref, Z_ref, q, G) - W[:, cols].astype(np.float64)) ** 2).reshape(K // G, G, -1).sum(axis=1)
    assert np.allclose(err.cpu().numpy()[:, cols], err_ref, rtol=1e-5, atol=1e-12)


@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("G", [64, 128, 256])
def test_columns_do_not_depend_on_the_launch(q, G):
    """The same columns in launches of one, two and four lanes a group (two and four at G = 256), also where weights are so far
    apart that their fp64 sums are rounded: 2^-60 to 1 in a column, and sums that decide between two codes."""
    K = 1024
    rng = np.random.default_rng(q + G)
    W = (rng.standard_normal((K, 64)) * 0.02).astype(np.float32)
    W[:, 8:32] = rng.uniform(1.0, 2.0, (K, 24)) * np.exp2(rng.integers(-60, 1, (K, 24))) * np.where(rng.random((K, 24)) < 0.5, -1, 1)
    W[:, 30] *= np.float32(2.0 ** -100)                                    # to where fp32 numbers are subnormal
    W[:, 31] *= np.float32(2.0 ** 120)
    W[:, 32:40] = np.where(rng.random((K, 8)) < 0.5, 0, W[:, 32:40])         # zeros are not far apart
    # two clusters with means 0 and 2 and a weight midway (equally near: code 0), unless the sum of the rest, -2^-50 each and
    # rounded away beside the others, is kept
    W[:, 40:48] = -2.0 ** -50
    W[:, 40:48].reshape(K // G, G, 8)[:, :11] = np.array([4, -1, 1] + 8 * [1.75], dtype=np.float32)[:, None]
    results = []
    for N in ((64, 2056) if G == 256 else (64, 2056, 16456)):
        wide = np.full((K, N), 0.01, dtype=np.float32)
        wide[:, :64], wide[:, -64:] = W, W
        codes, S, Z, err = (t.cpu().numpy() for t in B.hlq_quantize(B.make_desc(K, N, q, G), dev(wide), 3, with_err=True))
        for cols in (slice(0, 64), slice(N - 64, N)):
            results.append((codes[:, cols], S[:, :, cols].view(np.uint16), Z[:, cols].view(np.uint16), err[:, cols].view(np.uint32)))
    for other in results[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(results[0], other))
    if q == 1:
        codes = results[0][0][:, 40:48].reshape(K // G, G, 8)
        assert (codes[:, 2] == 0).all() and (codes[:, [0, 3]] == 1).all()
