"""hlq_quantize where its rounds end or its sorted lists are tested: parameters that stay as they are before the last round,
weights equal to a midpoint or next to one at zero, weights too far apart for exact sums, infinite weights beside finite ones."""
import functools

import numpy as np
import pytest

from oracle import hlq_quantize_oracle as QO
from paper_2510_19482_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


def quantize(W, q, G, rounds):
    return [t.cpu().numpy() for t in B.hlq_quantize(B.make_desc(*W.shape, q, G), dev(W), rounds)]


@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("G", [32, 64, 128, 256])
def test_rounds_after_the_last_change(q, G):
    # codes of the oracle after 2, 3, .. rounds; the columns of a wavefront come to rest after different numbers of them
    W = (np.random.default_rng(q * G).standard_normal((256, 136)) * 0.02).astype(np.float32)
    for rounds in (2, 3, 7, 40):
        assert np.array_equal(quantize(W, q, G, rounds)[0], QO.quantize(W.astype(np.float64), q, G, t_max=rounds)[0]), rounds
    # at rest, so the same bytes whatever is left (60 rounds and more suffice for these groups)
    a, b = quantize(W[:, :8], q, G, 300), quantize(W[:, :8], q, G, 301)
    assert all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(a, b))


@pytest.mark.parametrize("q", [1, 2, 3])
@pytest.mark.parametrize("G", [32, 64, 128])
def test_weights_at_the_midpoints(q, G):
    """First round only (the starting parameters are the same numbers on both sides, so are exact ties): a grid of 2^q + 1 steps
    whose ends make the candidates small integers, and weights at integers and halves, one fp32 step off them, and at zero from
    both sides."""
    rng = np.random.default_rng(5)
    W = np.empty((256, 72), dtype=np.float32)
    for n in range(72):
        low = np.float32(rng.integers(-8, 2))
        vals = low + rng.integers(0, 2 * (2 ** q - 1) + 1, 256) / np.float32(2)
        near = np.nextafter(vals.astype(np.float32), np.float32(rng.choice([-100, 100])))
        W[:, n] = np.where(rng.random(256) < 0.4, near, vals)
        W[::7, n] = rng.choice([0.0, -0.0, 1e-42, -1e-42, 2.0 ** -60, -2.0 ** -60], len(W[::7]))
        W[:, n] = np.clip(W[:, n], low, low + 2 ** q - 1)
        W[0::G, n], W[1::G, n] = low, low + 2 ** q - 1
    if G > 32:   # (far apart: rounded to what the sums hold, which the oracle does not do)
        W[np.abs(W) < 1e-10] = 0
    assert np.array_equal(quantize(W, q, G, 1)[0], QO.quantize(W.astype(np.float64), q, G, t_max=1)[0])


@pytest.mark.parametrize("q", [1, 2, 3, 4])
def test_groups_of_32_far_apart(q):
    # sums of such groups depend on the order: that of the rows, as fp64 sums of the oracle's design matrix have it up to rounding
    rng = np.random.default_rng(q)
    W = (rng.standard_normal((256, 136)) * 0.02).astype(np.float32)
    W[::5] *= np.float32(2.0 ** -30)
    W[3::32, ::2] = 0
    codes, S, Z = quantize(W, q, 32, 5)
    ref, S_ref, Z_ref = QO.quantize(W.astype(np.float64), q, 32, t_max=5)
    assert np.array_equal(codes, ref)
    # fp16 parameters: one unit in the last place (2^-10 of the value) and the subnormals' spacing
    for got, want in ((S, S_ref), (Z, Z_ref)):
        assert (np.abs(got.astype(np.float64) - want) <= 2.0 ** -10 * np.abs(want) + 2.0 ** -24).all()


@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("q", [1, 2, 3, 4])
def test_infinite_neighbours(q, G):
    # groups with infinities and NaN share wavefronts with finite ones, which keep their bytes
    W = (np.random.default_rng(9).standard_normal((256, 72)) * 0.02).astype(np.float32)
    alone = quantize(W, q, G, 4)
    W[5, 3], W[200, 40], W[130, 41], W[131, 41] = np.inf, np.nan, np.inf, -np.inf
    mixed = quantize(W, q, G, 4)
    keep = [n for n in range(72) if n not in (3, 40, 41)]
    for a, b in zip(alone, mixed):
        assert np.array_equal(np.ascontiguousarray(a[..., keep]).view(np.uint8), np.ascontiguousarray(b[..., keep]).view(np.uint8))


@pytest.mark.parametrize("rounds", [4, 5, 10, 30])
def test_lanes_of_groups_at_rest(rounds):
    """Four planes, groups of 64, enough columns for one lane a group: whole wavefronts, in which the last groups to change get two
    and four lanes, and an incomplete one (the last), in which they do not; with columns that are at rest at once, that scan, that have
    sums to be rounded."""
    K, N = 4096, 1032
    rng = np.random.default_rng(3)
    W = (rng.standard_normal((K, N)) * 0.02).astype(np.float32)
    W[:, 64:120] = 0.013
    W[:, 130] = (rng.integers(-1, 2, K) * 0.03).astype(np.float32)
    W[::3, 200] *= np.float32(2.0 ** -12)
    codes, S, Z = quantize(W, 4, 64, rounds)
    # (not the two with ties that are decided by how the parameters are rounded)
    cols = np.concatenate([np.arange(0, 64, 5), np.arange(118, 130), [131, 199, 201, 1023], np.arange(1024, 1032)])
    ref, S_ref, Z_ref = QO.quantize(W[:, cols].astype(np.float64), 4, 64, t_max=rounds)
    assert np.array_equal(codes[:, cols], ref)
    # fp16 parameters: one unit in the last place (2^-10 of the value) and the subnormals' spacing
    for got, want in ((S[:, :, cols], S_ref), (Z[:, cols], Z_ref)):
        assert (np.abs(got.astype(np.float64) - want) <= 2.0 ** -10 * np.abs(want) + 2.0 ** -24).all()


# columns of a wavefront that are not constant: as many as two lanes each suffice for, and fewer
LIVE = (32, 32, 30, 28, 24, 17)
LIVE_COLUMNS = np.concatenate([64 * b + np.arange(n) for b, n in enumerate(LIVE)])


@functools.lru_cache(maxsize=None)
def heavy_tailed():
    """Weights of six wavefronts by 16 groups of rows, and the oracle's codes and parameters of the live columns after every round."""
    K, q, G = 1024, 4, 64
    rng = np.random.default_rng(0)
    W = (rng.standard_normal((K, 64 * len(LIVE))) * 0.02).astype(np.float32)
    W[rng.random(W.shape) < 0.05] *= np.float32(20)
    Wg = QO.to_groups(W[:, LIVE_COLUMNS].astype(np.float64), G)
    s, z = QO.init_params(Wg, q)
    rounds = []
    for _ in range(9):
        codes = QO.select_bits(Wg, s, z, q)
        s, z = QO.lse(Wg, codes, s, z, q)
        rounds.append((codes, s, z))
    dead = np.setdiff1d(np.arange(W.shape[1]), LIVE_COLUMNS)
    W[:, dead] = 0.013
    return W, rounds


@pytest.mark.parametrize("rounds", [5, 6, 7, 8, 9])
def test_rounds_run_out_with_many_groups_changing(rounds):
    """The same kernel where the rounds end before it has come to 16 groups or fewer that change."""
    W, by_round = heavy_tailed()
    K, N = W.shape
    codes, S, Z = by_round[rounds - 1]
    # a group changes its parameters in a round where it has other codes than in the one before
    changing = (by_round[rounds - 2][0] != by_round[rounds - 3][0]).any(axis=1).reshape(K // 64, -1)
    start = np.concatenate([[0], np.cumsum(LIVE)])
    most = max(changing[:, a:b].sum(axis=1).max() for a, b in zip(start, start[1:]))
    assert most > 16 or rounds > 7, most
    wide = np.concatenate([W] + [W[:, :64]] * 28, axis=1)   # enough columns for one lane a group
    got = quantize(wide, 4, 64, rounds)
    assert np.array_equal(got[0][:, LIVE_COLUMNS], QO.from_groups_codes(codes, K, len(LIVE_COLUMNS), 64))
    # fp16 parameters: one unit in the last place (2^-10 of the value) and the subnormals' spacing
    for have, want in ((got[1], S.reshape(K // 64, -1, 4).transpose(2, 0, 1)), (got[2], Z.reshape(K // 64, -1))):
        assert (np.abs(have[..., LIVE_COLUMNS].astype(np.float64) - want) <= 2.0 ** -10 * np.abs(want) + 2.0 ** -24).all()
    # and every byte as by the launch of six wavefronts a group of rows, which has two lanes a group throughout
    for have, want in zip(got, quantize(W, 4, 64, rounds)):
        assert np.array_equal(np.ascontiguousarray(have[..., :N]).view(np.uint8), np.ascontiguousarray(want).view(np.uint8))
