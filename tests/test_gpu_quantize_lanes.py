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
