"""Grouped launches whose last column groups are cut along K: against the launch of the same call without (a workspace that
has no room for the partial sums) and against fp64."""
import pytest
import torch

from paper_2510_19482_amd import binding as B

from test_plan_tail import plan

pytestmark = pytest.mark.gpu
COUNTERS = 131072   # bytes ahead of the partial sums


def matrix(K, N, q, G, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    codes = torch.randint(0, 1 << q, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    scales = torch.randn((q, K // G, N), device="cuda", generator=g).mul_(0.02).abs_().half()
    zeros = torch.randn((K // G, N), device="cuda", generator=g).mul_(0.005).half()
    w = zeros.double().repeat_interleave(G, 0)
    for j in range(q):
        w += scales[j].double().repeat_interleave(G, 0) * (codes >> j & 1)
    return codes, scales, zeros, w


# row blocks of 128 x column groups of 256 columns just above 512, so that few of them are left for a second round;
# widths that end in part of a tile, 17 chunks (no even halves)
@pytest.mark.parametrize("q,G,M,shapes", [(2, 128, 1100, [(2048, 5000), (2048, 5000), (2048, 5064)]),
                                          (3, 64, 520, [(2176, 9224), (2176, 9224), (2176, 9480)]),
                                          (4, 32, 640, [(2048, 9224), (2048, 9480), (2048, 9224)])])
@pytest.mark.parametrize("f32", [False, True])
def test_cut_tail(q, G, M, shapes, f32):
    mats = [matrix(K, N, q, G, 7 * i + q) for i, (K, N) in enumerate(shapes)]
    descs = [B.make_desc(K, N, q, G) for K, N in shapes]
    packed = [B.hlq_pack(d, *m[:3]) for d, m in zip(descs, mats)]
    xs = {K: torch.randn((M, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(K)).half() for K, _ in shapes}
    X = [xs[K] for K, _ in shapes]
    out = [[torch.full((M, N), 7.0, dtype=torch.float32 if f32 else torch.float16, device="cuda") for _, N in shapes] for _ in range(2)]
    cut = B.GemmBatch(descs, packed, X, out[0], out_f32=f32)
    small = torch.zeros(cut.ws.numel() - 512, dtype=torch.uint8, device="cuda")
    whole = B.GemmBatch(descs, packed, X, out[1], out_f32=f32, ws=small)
    for launch in (cut, whole):
        launch.ws[COUNTERS:] = 0
        launch.launch()
        torch.cuda.synchronize()
        assert not launch.ws[:COUNTERS].any()
    # the part of the workspace that only the cut launch writes
    assert cut.ws[-4096:].any() and not small[-4096:].any()
    for (K, N), m, x, a, b in zip(shapes, mats, X, *out):
        ref = x.double() @ m[3]
        top = ref.abs().amax(dim=1, keepdim=True)
        # weights rounded to fp16 (2^-11 each, q + 1 times at most, over K terms of random sign) and fp16 results
        assert ((a.double() - ref).abs() / top).max() <= 1e-3
        # the two launches differ in the order of fp32 sums, and by that in the rounding of fp16 results
        assert ((a.double() - b.double()).abs() / top).max() <= (2e-6 if f32 else 1e-3)
        assert (a[:, :256] == b[:, :256]).all()   # never in the tail


# activations and results in wider matrices, results at addresses and strides of no more than their element's alignment; in the
# second set a problem that is in slices already beside the one whose tail is cut
@pytest.mark.parametrize("q,M,shapes,sliced", [(2, 1100, [(2048, 5000), (2048, 5000), (2048, 5064)], False),
                                               (3, 520, [(8192, 2056), (2048, 9224), (2048, 9736)], True)])
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("big", [False, True])
def test_strides_slices_and_range(q, M, shapes, sliced, f32, big):
    """big: scales of 700 and 3000 in the last column that is cut and in the first problem, for which the call is computed again."""
    cut, slices = plan(shapes, q, M)
    assert cut is not None and (max(slices) > 1) == sliced
    mats = []
    for i, (K, N) in enumerate(shapes):
        codes, scales, zeros, w = matrix(K, N, q, 128, 11 * i + q)
        if big and i in (0, cut[0]):
            at = scales[0, 1, N - 1].clone()
            scales[0, 1, N - 1] = 3000.0 if i else 700.0
            w[128:256, N - 1] += (scales[0, 1, N - 1].double() - at.double()) * (codes[128:256, N - 1] & 1)
        mats.append((codes, scales, zeros, w))
    descs = [B.make_desc(K, N, q, 128) for K, N in shapes]
    packed = [B.hlq_pack(d, *m[:3]) for d, m in zip(descs, mats)]
    X = [torch.randn((M, K + 24), device="cuda", generator=torch.Generator(device="cuda").manual_seed(K + i)).half()[:, 16:16 + K] for i, (K, _) in enumerate(shapes)]
    wide = [torch.full((M, N + 7), 7.0, dtype=torch.float32 if f32 else torch.float16, device="cuda") for _, N in shapes]
    Y = [w[:, 3:3 + N] for w, (_, N) in zip(wide, shapes)]
    batch = B.GemmBatch(descs, packed, X, Y, out_f32=f32)
    for _ in range(2):
        batch.launch()
        torch.cuda.synchronize()
        assert not batch.ws[:COUNTERS].any()
    for (K, N), m, x, y, w in zip(shapes, mats, X, Y, wide):
        assert (w[:, :3] == 7).all() and (w[:, 3 + N:] == 7).all()
        ref = x.double() @ m[3]
        # as above; where the call is computed again its weights are exact, and fp16 results that are too large are infinite
        finite = y.isfinite()
        assert finite.all() or (big and not f32 and (ref.abs()[~finite] > 65500).all())
        for part in (slice(0, N - 1), slice(N - 1, N)):   # (the last column may be the one with the large scale)
            err = torch.where(finite, (y.double() - ref).abs(), 0.0)[:, part]
            assert err.max() <= 1e-3 * ref[:, part].abs().max()


def test_replays():
    """The cut launch and its sums in a graph, replayed after eager work on the same workspace."""
    q, G, M, shapes = 2, 128, 1100, [(2048, 5000), (2048, 5000), (2048, 5064)]
    mats = [matrix(K, N, q, G, i) for i, (K, N) in enumerate(shapes)]
    descs = [B.make_desc(K, N, q, G) for K, N in shapes]
    X = torch.randn((M, 2048), device="cuda").half()
    Y = [torch.empty((M, N), dtype=torch.float16, device="cuda") for _, N in shapes]
    batch = B.GemmBatch(descs, [B.hlq_pack(d, *m[:3]) for d, m in zip(descs, mats)], [X] * 3, Y)
    batch.launch()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        batch.launch()
    for i in range(3):
        X.copy_(torch.randn((M, 2048), device="cuda").half())
        graph.replay()
        torch.cuda.synchronize()
        got = [y.clone() for y in Y]
        batch.launch()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, Y))
