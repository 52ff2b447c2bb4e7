"""Grouped launches whose last column groups are cut along K: the plan, as the workspace query shows it, against a model of the launch
that knows every one of its 512 places."""
import ctypes
import random

import pytest

from paper_2510_19482_amd import binding as B

COUNTERS = 131072


def ceil(a, b):
    return -(-a // b)


def end(kinds):
    """When the last workgroup ends: kinds of workgroups (steps, number) in the order of the launch, each to the place with the least to do;
    then the longest shares a unit with the shortest, and runs at 1 / 0.6 the speed once it is alone."""
    places = {0: 512}
    for steps, number in kinds:
        while number:
            low = min(places)
            taken = min(number, places[low])
            number -= taken
            places[low] -= taken
            if not places[low]:
                del places[low]
            places[low + steps] = places.get(low + steps, 0) + taken
            if len(places) > 48:
                return None
    loads = sorted(load for load, n in places.items() for _ in range(n))
    return max(loads[i] + 0.6 * (loads[511 - i] - loads[i]) for i in range(256))


def plan(shapes, q, M):
    """(problem, column groups, chunks a slice, slices) of the part that is cut; slices of the problems; row blocks of 128"""
    rows = ceil(M, 128)
    chunks, groups = [ceil(K, 128) for K, _ in shapes], [ceil(N, 256) for _, N in shapes]
    target = max(2, int(sum(float(g) * rows * c for g, c in zip(groups, chunks)) / 512 + 0.999))
    cps, slices = [], []
    for c in chunks:
        cps.append(ceil(ceil(c, max(1, ceil(c, target))), 2) * 2)
        slices.append(ceil(c, cps[-1]))
    number = [g * rows * s for g, s in zip(groups, slices)]
    whole = [i for i, s in enumerate(slices) if s == 1]
    if not 512 < sum(number) <= 4096 or not whole:
        return None, slices
    wide = min(whole, key=lambda i: (chunks[i], -ceil(shapes[i][1], 64), i))
    order = sorted(range(len(shapes)), key=lambda i: -cps[i])
    uncut = end([(cps[i], number[i]) for i in order])
    if chunks[wide] < 16 or uncut is None:
        return None, slices
    step, best, cut = 3.0 + 0.3 * q, uncut * (3.0 + 0.3 * q) * 0.96, None
    for c in range(1, groups[wide], 1 + groups[wide] // 16):
        for ns in (2, 3):
            if c * rows > 256:
                continue
            length = ceil(ceil(chunks[wide], ns), 2) * 2
            steps = end([(cps[i], number[i] - (c * rows if i == wide else 0)) for i in order] + [(length, c * rows * ns)])
            if steps is None:
                continue
            t = steps * step + (0.0 if max(slices) > 1 else 5.0) + c * rows * ns * (128 * 256 * 4) / 4.0e6
            if t < best:
                best, cut = t, (wide, c, length, ceil(chunks[wide], length))
    return cut, slices


def query(shapes, q, M):
    descs = (B.HlqDesc * len(shapes))(*[B.make_desc(K, N, q, 128) for K, N in shapes])
    n = ctypes.c_size_t()
    assert B.lib.hlq_gemm_batch_workspace_bytes(len(shapes), descs, M, ctypes.byref(n)) == 0
    return n.value


def check(shapes, q, M):
    shapes = sorted(shapes, key=lambda s: -ceil(s[0], 128))
    cut, slices = plan(shapes, q, M)
    one_by_one = COUNTERS + sum(B.workspace_bytes(B.make_desc(K, N, q, 128), M) - COUNTERS for K, N in shapes)
    grouped = COUNTERS + sum(s * M * N * 4 for s, (_, N) in zip(slices, shapes) if s > 1)
    if cut:
        i, groups, _, ns = cut
        grouped += ns * M * (shapes[i][1] - (ceil(shapes[i][1], 256) - groups) * 256) * 4
    assert query(shapes, q, M) == ceil(max(one_by_one, grouped), 256) * 256, (shapes, q, M, cut)
    return cut


# places of two loads that are as many as each other: they run out together, and what is left is paired with what is left
@pytest.mark.parametrize("shapes,q,M,cut", [([(5504, 18680), (5248, 18016)], 4, 2048, None), ([(6784, 16504), (6784, 11936)], 2, 2048, None),
                                            ([(4224, 10128), (3968, 11256)], 3, 2048, (1, 4, 12, 3)), ([(7936, 14984), (7936, 13328)], 3, 1024, (0, 17, 32, 2)),
                                            ([(4608, 11200), (2944, 6776)], 2, 1000, (1, 1, 12, 2)), ([(5632, 10192), (4224, 8192)], 1, 1500, (1, 7, 12, 3))])
def test_loads_that_run_out_together(shapes, q, M, cut):
    assert check(shapes, q, M) == cut


def test_plans_of_many_launches():
    rng = random.Random(1)
    for _ in range(300):
        shapes = [(128 * rng.randint(16, 64), 8 * rng.randint(400, 2500)) for _ in range(rng.randint(2, 7))]
        if rng.random() < 0.5:
            shapes = [(shapes[0][0], N) for _, N in shapes]
        check(shapes, rng.randint(1, 4), rng.choice([128, 256, 512, 640, 1024, 1536, 2048]))


def test_the_layer_of_the_benchmark():
    layer = [(4096, 4096), (4096, 1024), (4096, 1024), (4096, 4096), (4096, 14336), (4096, 14336), (14336, 4096)]
    assert check(layer, 2, 512) == (5, 9, 16, 2)
    assert check(layer, 2, 2048) is None
