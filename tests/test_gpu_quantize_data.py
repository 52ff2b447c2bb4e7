"""hlq_quantize on weights as checkpoints have them -- rounded to 16 bits, on a coarse grid, with dead columns -- where
candidate midpoints fall on zero and candidates coincide: the codes against the oracle, and the time against that of fp32
normals (it does not depend on the data by more than the bound beside each case)."""
import numpy as np
import pytest
import torch

from oracle import hlq_quantize_oracle as QO
from paper_2510_19482_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


def weights(kind, K, N):
    rng = np.random.default_rng(11)
    W = (rng.standard_normal((K, N)) * 0.02).astype(np.float32)
    if kind == "bf16":
        W = (((W.view(np.uint32) + 0x8000) >> 16) << 16).view(np.float32)
        W[0::32], W[1::32] = W[2::32] * 4, -W[2::32] * 4     # many groups with min = -max: a midpoint at zero
    if kind == "dead":
        W[:, 7::64] = 0.0
        W[:, 9::64] = 0.013
    if kind == "mixed":
        W[:, 7::64] = (rng.integers(-1, 2, (K, N))[:, 7::64] * 0.03).astype(np.float32)
    if kind == "ternary":
        W = (rng.integers(-1, 2, (K, N)) * 0.03).astype(np.float32)
    if kind == "steps":
        W = (rng.integers(-8, 8, (K, N)) * 0.003).astype(np.float32)
    return W


def microseconds(q, G, W):
    d = B.make_desc(*W.shape, q, G)
    best = float("inf")
    for _ in range(6):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(10):
            B.hlq_quantize(d, W, 10)
        stop.record()
        stop.synchronize()
        best = min(best, start.elapsed_time(stop) * 100)
    return best


# every format once; 1 round (the starting parameters are the same numbers on both sides, so are exact ties), then 10
@pytest.mark.parametrize("kind,rounds", [("bf16", 1), ("bf16", 10), ("dead", 1), ("dead", 10), ("ternary", 1), ("steps", 1)])
@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("G", [32, 64, 128, 256])
def test_codes(kind, rounds, q, G):
    W = weights(kind, 512, 72)
    codes, _, _ = B.hlq_quantize(B.make_desc(512, 72, q, G), dev(W), rounds)
    assert np.array_equal(codes.cpu().numpy(), QO.quantize(W.astype(np.float64), q, G, t_max=rounds)[0])


# one column in 64 needs the scan in every round and takes the others, whose weights are all different, along
@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("G", [32, 64, 128, 256])
@pytest.mark.parametrize("rounds", [1, 10])
def test_codes_beside_a_column_of_few_values(rounds, q, G):
    W = weights("mixed", 512, 72)
    codes = B.hlq_quantize(B.make_desc(512, 72, q, G), dev(W), rounds)[0].cpu().numpy()
    ref = QO.quantize(W.astype(np.float64), q, G, t_max=rounds)[0]
    normal = np.arange(72) % 64 != 7   # (after the first round the others' ties are decided by how the parameters are rounded)
    assert np.array_equal(codes[:, normal], ref[:, normal])
    assert rounds > 1 or np.array_equal(codes, ref)


# bound: what was measured, and a quarter more; with a scan of all candidates from memory for these the ratios were
# 1.7, 1.3, 1.4, 5.5, 2.2, 5.5 and 3.8; "mixed" run by run of equal weights 5.3, 4.2 and 3.8
@pytest.mark.parametrize("kind,q,G,bound", [("bf16", 1, 128, 1.3), ("bf16", 2, 64, 1.3), ("bf16", 1, 256, 1.25),
                                           ("dead", 2, 128, 1.25), ("dead", 4, 32, 1.25), ("ternary", 2, 128, 2.0),
                                           ("ternary", 4, 128, 2.6), ("mixed", 2, 64, 3.1), ("mixed", 3, 128, 3.3), ("mixed", 2, 32, 2.5)])
def test_time_does_not_depend_on_the_data(kind, q, G, bound):
    plain, special = (microseconds(q, G, dev(weights(k, 4096, 4096))) for k in ("plain", kind))
    print(kind, q, G, f"{special:.1f} us, fp32 normals {plain:.1f} us", flush=True)
    assert special <= bound * plain


@pytest.mark.parametrize("q", [1, 2, 3])
@pytest.mark.parametrize("kind", ["bf16", "steps"])
def test_small_launch(q, kind):
    # one wavefront per SIMD, groups of 32
    plain, special = (microseconds(q, 32, dev(weights(k, 1024, 1024))) for k in ("plain", kind))
    print(kind, q, f"{special:.1f} us, fp32 normals {plain:.1f} us", flush=True)
    assert special <= 1.18 * plain
