"""Work split of launches of several rows, on the host: the run length is chosen per launch, and neither the choice nor the
limits of the counter block and of the block arithmetic may refuse what a fixed run length was accepted for."""
import pytest

from paper_2510_19482_amd import binding as B

from test_plan_host import check_plan


# K and N at both ends of their range, ragged tiles, odd numbers of chunks; short runs on K = 2^21 with eight thousand columns or
# N = 2^20 take more slices than the block arithmetic or the counter block has room for
@pytest.mark.parametrize("K,N", [(512, 512), (128 * 67, 5000), (4096, 14336), (14336, 4096), (128 * 33, 128256), (8192, 131072),
                                 (1 << 21, 8), (1 << 21, 8192), (256, 1 << 20), (4096, 1 << 20)])
@pytest.mark.parametrize("G,M", [(32, 2), (64, 2), (64, 4), (128, 2), (128, 4), (128, 8), (256, 16)])
@pytest.mark.parametrize("count", [1, 3, 8])
def test_runs_of_every_launch_fit(K, N, G, M, count):
    if K % G:
        pytest.skip("K is no multiple of the group")
    for q in (1, 4):
        infos = B.gemv_plan_query([B.make_desc(K, N, q, G)] * count, M)
        at = 0
        for info in infos:
            check_plan(info, K // 128, (K, N, q, G, M, count))
            assert info.first_block == at
            at += info.blocks


def test_run_follows_the_rounds_of_the_launch():
    # 24 and 64 chunks: one round of 512 workgroups with six chunks a wavefront, not two of four
    layer = [(3072, 3072)] * 2 + [(3072, 512)] * 2 + [(3072, 8192)] * 2 + [(8192, 3072)]
    infos = B.gemv_plan_query([B.make_desc(K, N, 4, 128) for K, N in layer], 8)
    assert sum(i.blocks for i in infos) == 512
    assert max(-(-i.chunks_per_slice // i.waves_per_tile) for i in infos) == 6


def test_rows_beyond_the_kernels_have_no_plan():
    # three rows at G = 32 exceed the two row sets of the 64-column kernel: only the launches that the 16-column kernel takes
    # (256 to 4096 chunk-tiles of at most 64 chunks, or 14000 and more) have a plan
    for K, N, planned in [(512, 512, False), (4096, 4096, True), (4096, 14336, False), (8192, 16384, True)]:
        descs = [B.make_desc(K, N, 2, 32)]
        if planned:
            assert B.gemv_plan_query(descs, 3)[0].blocks > 0
        else:
            with pytest.raises(B.HlqError):
                B.gemv_plan_query(descs, 3)


# a forced plan changes how K is cut and nothing else: two to four rows that go to the 16-column kernel, whose workgroups own
# fewer columns than a tile has, are planned whatever is forced
@pytest.mark.parametrize("W,cpw", [(0, 1), (1, 1), (1, 2), (1, 100), (2, 1), (4, 2), (8, 1), (8, 100), (16, 3), (0, 5000)])
@pytest.mark.parametrize("K,N,G,M,count", [(640, 557248, 32, 2, 4), (14080, 845040, 64, 4, 1), (1 << 17, 8192, 32, 3, 8), (1 << 20, 131072, 64, 3, 1),
                                           (1 << 21, 16384, 32, 4, 1), (512, 1 << 20, 64, 3, 8), (128, 1 << 20, 32, 2, 1), (4096, 4096, 128, 4, 1)])
def test_forced_plans_refuse_nothing(K, N, G, M, count, W, cpw):
    descs = [B.make_desc(K, N, 1, G)] * count
    B.set_gemv_plan(0, W, cpw)
    try:
        infos = B.gemv_plan_query(descs, M)
    finally:
        B.set_gemv_plan(0, 0, 0)
    for info in infos:
        check_plan(info, K // 128, (K, N, G, M, count, W, cpw))
    # partial results of a workgroup: 64 bytes per row of four (two) and column block and wavefront on it, beside its operands
    blocks = -(-(-(-N // 16)) // infos[0].tile_groups)
    rows = 2 if M == 2 else 4
    assert blocks * infos[0].waves_per_tile * 64 * rows + infos[0].waves_per_workgroup * 6400 <= 160 * 1024


# the same of the few-rows kernel, whose own choice of four wavefronts a workgroup would double the slices of a forced run
@pytest.mark.parametrize("K,N,G,count,cpw", [(128 * 9921, 922440, 128, 1, 3), (1174528, 76184, 128, 4, 1), (992256, 100424, 256, 1, 1)])
def test_forced_runs_of_the_few_rows_kernel(K, N, G, count, cpw):
    B.set_gemv_plan(0, 0, cpw)
    try:
        infos = B.gemv_plan_query([B.make_desc(K, N, 3, G)] * count, 2)
    finally:
        B.set_gemv_plan(0, 0, 0)
    for info in infos:
        check_plan(info, K // 128, (K, N, G, count, cpw))


# two to four rows on the 16-column kernel only where a wavefront walks over enough columns with the operands that it makes
@pytest.mark.parametrize("K,N,G,M,columns", [(256, 65536, 128, 2, False), (512, 4096, 128, 3, False), (8192, 256, 64, 4, False), (6144, 5120, 256, 2, False),
                                             (28672, 24576, 64, 3, False), (8192, 14336, 32, 2, False), (2048, 6144, 128, 4, True), (4096, 1024, 64, 2, True),
                                             (8192, 4096, 128, 4, True), (4096, 28672, 64, 4, True), (8192, 18432, 64, 3, True), (28672, 24576, 32, 4, True)])
def test_two_to_four_rows_by_columns(K, N, G, M, columns):
    info = B.gemv_plan_query([B.make_desc(K, N, 2, G)], M)[0]
    tiles = -(-(-(-N // 64)) // (info.waves_per_workgroup // info.waves_per_tile))   # workgroups that own whole tiles
    assert (info.tile_groups != tiles) == columns
