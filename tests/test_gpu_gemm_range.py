"""Scales outside the range of the fp16 rebuild of the tiled kernel (|s| >= 512): the call is computed again in fp32, by a
kernel of its own behind calls whose K is not split and by the one that adds the partial sums behind the others."""
import numpy as np
import pytest
import torch

from oracle import c_oracle
from oracle import hlq_oracle as O
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth

from gpu_util import TOL, dev, pack_on_gpu

pytestmark = pytest.mark.gpu

COUNTER_BYTES = 131072


def group(shapes, M, q=2, G=64, big=0):
    """Batch of problems, the one with index `big` with one scale of 3000, and the reference products."""
    descs, packed, Xs, refs = [], [], [], []
    for i, (K, N) in enumerate(shapes):
        codes, S, Z = synth.make_weight(K, N, q, G, "range", i)
        if i == big:
            S = S.copy()
            S[0, 1, N - 3] = np.float16(3000.0)
        X = synth.make_x(M, K, "range", i)
        d, p = pack_on_gpu(codes, S, Z, q, G)
        descs.append(d)
        packed.append(p)
        Xs.append(dev(X))
        refs.append(c_oracle.gemm_f64(X, codes, S, Z, q, G))
    ys = [torch.full((M, N), 7.0, dtype=torch.float32, device="cuda") for _, N in shapes]
    return B.GemmBatch(descs, packed, Xs, ys, out_f32=True), ys, refs


def check(batch, ys, refs):
    for _ in range(2):      # the flag and the count are lowered again by each call
        for y in ys:
            y.fill_(7.0)
        batch.launch()
        for y, ref in zip(ys, refs):
            assert O.row_rel_err(y.cpu().numpy().astype(np.float64), ref).max() <= TOL
        assert int(batch.ws[:COUNTER_BYTES].count_nonzero()) == 0


@pytest.mark.parametrize("M", [17, 40, 70])
def test_calls_that_split_nothing(M):
    # K of two chunks cannot be split: the recomputation has a launch of its own
    check(*group([(256, 328)], M))
    check(*group([(256, 200), (256, 1096), (128, 72)], M, big=1))


def microseconds(batch):
    best = float("inf")
    for _ in range(4):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(4):
            batch.launch()
        stop.record()
        stop.synchronize()
        best = min(best, start.elapsed_time(stop) * 250)
    return best


def test_group_that_splits_a_narrow_problem_only():
    # The sums are one workgroup's work here; the 1285 items of the second computation are not.  By the narrow problem's own
    # wavefronts alone the group takes some twenty times as long as that problem, whose five items are the longest.
    M, narrow, wide = 40, (4096, 8), (256, 16384)
    both, alone = group([narrow, wide], M), group([narrow, narrow], M)
    check(*both)
    t, t_alone = microseconds(both[0]), microseconds(alone[0])
    print(f"{t:.0f} us, the narrow problem {t_alone:.0f} us", flush=True)
    assert t <= 4 * t_alone
