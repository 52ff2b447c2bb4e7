"""The one-row matrix-core kernel with 16 columns x 4 chunks per wavefront (hlq_gemv_cols.hip) at its edges: narrow tiles
and half column blocks, windows with missing chunks, one step and several per wavefront, two K slices (exchange per column)
and more (partial sums), both sides of the size rule that sends a launch there."""
import numpy as np
import pytest
import torch

from oracle import c_oracle
from oracle import hlq_oracle as O
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth

from gpu_util import dev, pack_on_gpu

pytestmark = pytest.mark.gpu

# fp32 results: the matrix core keeps 13 bits below the largest product of a run of eight
TOL_F32 = 2e-4


@pytest.fixture(autouse=True)
def auto_plan():
    B.set_gemv_path(B.GEMV_MX)
    yield
    B.set_gemv_plan(0, 0, 0)
    B.set_gemv_path(B.GEMV_AUTO)


def case(K, N, q, G, *key):
    codes, S, Z = synth.make_weight(K, N, q, G, "cols", *key)
    x = synth.make_x(1, K, "cols", K, N, *key, outliers=True)
    d, packed = pack_on_gpu(codes, S, Z, q, G)
    return d, packed, dev(x[0]), c_oracle.gemm_f64(x, codes, S, Z, q, G)


def check(y, ref):
    assert O.row_rel_err(y.cpu().numpy().astype(np.float64)[None, :], ref).max() <= TOL_F32


# K: one chunk, part of a window, a window and a chunk, 8 and 9 windows, 16 and 17 windows (two slices), 33 (three slices)
@pytest.mark.parametrize("K,N", [(256, 8), (384, 24), (640, 72), (1280, 136), (4096, 1000), (4608, 40), (8192, 88),
                                 (8704, 200), (16384, 56), (16896, 72)])
@pytest.mark.parametrize("q,G", [(1, 128), (2, 64), (2, 256), (3, 32), (4, 32), (4, 128)])
def test_edges(K, N, q, G):
    K = -(-K // G) * G
    d, packed, x, ref = case(K, N, q, G)
    ws = B.alloc_workspace(d, 1)
    info = B.gemv_plan_query([d], 1)[0]
    print("cols", K, N, q, G, "slices", info.slices, "groups", info.tile_groups, flush=True)
    y = torch.full((N,), 7.0, dtype=torch.float32, device="cuda")
    first = None
    for _ in range(3):      # the workspace is left as it was found, the order of the sums is fixed
        y.fill_(7.0)
        B.hlq_lut_gemv(d, packed, x, y, out_f32=True, ws=ws)
        check(y, ref)
        first = y.clone() if first is None else first
        assert torch.equal(y, first)


@pytest.mark.parametrize("W,cpw", [(1, 1), (2, 5), (4, 2), (8, 9), (16, 1), (16, 3)])
@pytest.mark.parametrize("q,G", [(2, 128), (3, 64), (2, 256)])
def test_forced_splits(W, cpw, q, G):
    K, N = 4864, 1096       # 38 chunks, a tail of 8 columns
    B.set_gemv_plan(0, W, cpw)
    d, packed, x, ref = case(K, N, q, G, "forced")
    check(B.hlq_lut_gemv(d, packed, x, out_f32=True), ref)


def test_two_slices_of_several_problems_share_one_counter_block():
    q, G = 2, 128
    shapes = [(14336, 2048), (9216, 1032), (16384, 8), (4096, 520)]
    cases = [case(K, N, q, G, "pairs") for K, N in shapes]
    ys = [torch.empty(N, dtype=torch.float32, device="cuda") for _, N in shapes]
    infos = B.gemv_plan_query([c[0] for c in cases], 1)
    assert [i.slices for i in infos] == [2, 2, 2, 1]
    batch = B.GemvBatch([c[0] for c in cases], [c[1] for c in cases], [c[2] for c in cases], ys, out_f32=True)
    for _ in range(3):
        for y in ys:
            y.fill_(7.0)
        batch.launch()
        for c, y in zip(cases, ys):
            check(y, c[3])
    assert int(batch.ws[:131072].count_nonzero()) == 0


def test_counters_and_slots_side_by_side():
    # three slices with an odd number of arrival counters in front of two slices with 64-bit slots
    q, G = 2, 128
    shapes = [(16896, 72), (14336, 40), (12288, 24)]
    cases = [case(K, N, q, G, "mixed") for K, N in shapes]
    ys = [torch.empty(N, dtype=torch.float32, device="cuda") for _, N in shapes]
    infos = B.gemv_plan_query([c[0] for c in cases], 1)
    assert [i.slices for i in infos] == [3, 2, 2] and infos[0].tile_groups % 2 == 1
    batch = B.GemvBatch([c[0] for c in cases], [c[1] for c in cases], [c[2] for c in cases], ys, out_f32=True)
    for _ in range(3):
        for y in ys:
            y.fill_(7.0)
        batch.launch()
        for c, y in zip(cases, ys):
            check(y, c[3])
    assert int(batch.ws[:131072].count_nonzero()) == 0


def is_cols(d):
    """Whether a one-row launch goes to the 16-column kernel: with K = 4096 its plan has eight wavefronts on a column block,
    and a workgroup per share of ceil(N / 16) blocks; the 64-column kernel has one per W / kw tiles."""
    i = B.gemv_plan_query([d], 1)[0]
    tiles, per = -(-d.N // 64), i.waves_per_workgroup // i.waves_per_tile
    return i.tile_groups != -(-tiles // per)


# K = 4096: 32 chunk-tiles per 64 columns.  first: the first N (a multiple of 64) whose launch is at or past the named
# number of chunk-tiles
@pytest.mark.parametrize("q,G,units,below", [(2, 32, 12000, True), (4, 32, 12000, True), (2, 64, 60000, True), (3, 64, 60000, True),
                                             (1, 64, 20000, True), (1, 128, 20000, True), (1, 128, 60000, False)])
def test_either_side_of_the_size_rule(q, G, units, below):
    first = -(-units // 32) * 64
    for n, cols in ((first - 64, below), (first - 40, not below)):      # 40 columns of one more tile
        d, packed, x, ref = case(4096, n, q, G, "rule")
        assert is_cols(d) == cols, n
        check(B.hlq_lut_gemv(d, packed, x, out_f32=True), ref)
