"""Edges of the offline kernels: hlq_pack on code tensors at any byte address and tile widths from 8 to 64 against the
layout written out in numpy, and the quantizer's bit-pattern selection on data full of exact ties."""
import numpy as np
import pytest
import torch

from oracle import hlq_quantize_oracle as QO
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth

from gpu_util import dev

pytestmark = pytest.mark.gpu


def layout(codes, S, Z, q, G):
    """The packed blob: tiles of 64 columns, records of 128 k: planes (16 bytes a column), then the scales and zeros of
    the groups that start in the record; bit (k >> 1) + 16 (k & 1) of a 32-bit word is weight k of its block."""
    K, N = codes.shape
    out = []
    for n0 in range(0, N, 64):
        cols = slice(n0, min(n0 + 64, N))
        for k0 in range(0, K, 128):
            blk = codes[k0:k0 + 128, cols].astype(np.uint64).reshape(4, 32, -1)
            for j in range(q):
                w = np.zeros((4, blk.shape[2]), dtype=np.uint64)
                for k in range(32):
                    w |= ((blk[:, k] >> np.uint64(j)) & np.uint64(1)) << np.uint64((k >> 1) + 16 * (k & 1))
                out.append(np.ascontiguousarray(w.T.astype(np.uint32)).tobytes())
            for g in range(-(-k0 // G), -(-(k0 + 128) // G)):
                out += [S[j, g, cols].tobytes() for j in range(q)] + [Z[g, cols].tobytes()]
    return np.frombuffer(b"".join(out), dtype=np.uint8)


@pytest.mark.parametrize("offset", [0, 1, 2, 4])
@pytest.mark.parametrize("K,N,q,G", [(128, 8, 1, 32), (256, 72, 2, 64), (384, 264, 3, 128), (512, 56, 4, 256), (256, 320, 4, 32)])
def test_pack_layout_at_any_address(K, N, q, G, offset):
    codes, S, Z = synth.make_weight(K, N, q, G, "packedge")
    d = B.make_desc(K, N, q, G)
    buf = torch.zeros(K * N + 16, dtype=torch.uint8, device="cuda")
    buf[offset:offset + K * N] = dev(codes).reshape(-1)
    packed = B.hlq_pack(d, buf[offset:offset + K * N].view(K, N), dev(S), dev(Z))
    assert np.array_equal(packed.cpu().numpy(), layout(codes, S, Z, q, G))


@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("G", [32, 64, 128, 256])
def test_selection_on_ties(q, G):
    # weights on a coarse symmetric grid: candidate midpoints fall on weights, on zero, and coincide.  One round: the
    # starting parameters are the same numbers on both sides, so the codes have to be the same everywhere.
    K, N = 512, 72
    rng = np.random.default_rng(7 * q + G)
    W = (rng.integers(-12, 13, (K, N)) / 8.0).astype(np.float32)
    W[0::G], W[1::G] = 1.5, -1.5                     # the grid's midpoint is exactly zero
    W[:, 40:] *= np.float32(2.0 ** -140)             # and in the subnormal range of fp32 (multiples of 2^-143)
    W[:, 64:] = rng.integers(0, 2, (K, 8)).astype(np.float32)   # all candidates but two unused
    W[:, 70] = 0.25                                  # equal candidates
    codes_ref, _, _ = QO.quantize(W.astype(np.float64), q, G, t_max=1)
    codes, _, _ = B.hlq_quantize(B.make_desc(K, N, q, G), dev(W), 1)
    assert np.array_equal(codes.cpu().numpy(), codes_ref)
