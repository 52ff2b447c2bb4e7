"""The kernel for up to 32 rows that cuts K inside a workgroup (hlq_gemm_short.hip): wavefronts without a chunk, odd chunk
counts, narrow and single tiles, both sizes of row block at their edges, K slices, strided rows, parameters out of range."""
import numpy as np
import pytest
import torch

from oracle import hlq_oracle as O
from paper_2510_19482_amd import binding as B
from paper_2510_19482_amd import synth

from gpu_util import dev, pack_on_gpu

pytestmark = pytest.mark.gpu

F32_TOL = 1e-3   # weights rounded to fp16 when rebuilt (2^-11 each), of a row's largest result


def run(K, N, q, G, M, key, scale=1.0, pad=0):
    codes, S, Z = synth.make_weight(K, N, q, G, "short", key)
    S, Z = (S * np.float16(scale)).astype(np.float16), (Z * np.float16(scale)).astype(np.float16)
    X = synth.make_x(M, K, "short", key, outliers=True)
    desc, packed = pack_on_gpu(codes, S, Z, q, G)
    xbuf = torch.full((M, K + 8 * pad), float("nan"), dtype=torch.float16, device="cuda")
    xbuf[:, :K] = dev(X)
    ybuf = torch.full((M, N + 4 * pad), 7.0, dtype=torch.float32, device="cuda")
    ws = B.alloc_workspace(desc, M)
    for _ in range(2):   # the second call finds the workspace as the first one left it
        B.hlq_lut_gemm(desc, packed, xbuf[:, :K], ybuf[:, :N], out_f32=True, ws=ws)
    Y = ybuf.cpu().numpy().astype(np.float64)
    if pad:
        assert (Y[:, N:] == 7.0).all()
    assert O.row_rel_err(Y[:, :N], O.gemm_dequant(X, codes, S, Z, q, G)).max() <= F32_TOL
    return ws


@pytest.mark.parametrize("M", [5, 16, 17, 32])
@pytest.mark.parametrize("q,G", [(1, 32), (2, 64), (3, 64), (4, 32), (2, 256), (4, 128)])
def test_row_blocks_and_formats(q, G, M):
    run(2304 if G < 256 else 2560, 200, q, G, M, "formats")   # 18 or 20 chunks for eight wavefronts, a last tile of 8 columns


@pytest.mark.parametrize("K,N", [(128, 8), (128, 64), (256, 136), (1152, 72), (3968, 64)])
def test_few_chunks(K, N):
    run(K, N, 3, 64, 19, "few")


@pytest.mark.parametrize("M", [6, 24])
@pytest.mark.parametrize("scale", [1.0, 30000.0])   # times N(0, 0.02): most scales beyond 512 are met in every tile
def test_slices_strides_and_range(M, scale):
    """4096 x 512: K in four slices; 1024 x 16448: none (257 tiles)."""
    run(4096, 512, 2, 64, M, "sliced", scale, pad=2)
    ws = run(1024, 16448, 2, 64, M, "whole", scale, pad=1)
    assert int(ws[:131072].view(torch.int32).abs().sum()) == 0   # flags and counters are left cleared


def test_one_tile_out_of_range():
    """A parameter out of range changes how its own tile is computed, no other."""
    K, N, q, G, M = 1024, 16448, 3, 64, 9
    codes, S, Z = synth.make_weight(K, N, q, G, "short", "one")
    X = synth.make_x(M, K, "short", "one")
    S[0, 3, 70] = 60000.0
    desc, packed = pack_on_gpu(codes, S, Z, q, G)
    Y = B.hlq_lut_gemm(desc, packed, dev(X), out_f32=True).cpu().numpy().astype(np.float64)
    ref = O.gemm_dequant(X, codes, S, Z, q, G)
    # column by column: the one column is 1e6 times the others
    assert (np.abs(Y - ref).max(0) <= F32_TOL * np.maximum(np.abs(ref).max(0), np.median(np.abs(ref).max(0)))).all()
    assert (np.abs(Y - ref)[:, 64:128].max(0) <= 2e-5 * np.abs(ref[:, 64:128]).max(0)).all()


@pytest.mark.parametrize("M", [7, 21])
def test_grouped_launch(M):
    q, G = 2, 64
    shapes = [(1024, 520), (4096, 200), (256, 64), (896, 8), (2048, 1096)]
    descs, packs, Xs, Ys, refs, bounds = [], [], [], [], [], []
    for i, (K, N) in enumerate(shapes):
        codes, S, Z = synth.make_weight(K, N, q, G, "short-group", i)
        X = synth.make_x(M, K, "short-group", i)
        d, p = pack_on_gpu(codes, S, Z, q, G)
        descs.append(d); packs.append(p); Xs.append(dev(X))
        Ys.append(torch.zeros((M, N), dtype=torch.float32, device="cuda"))
        refs.append(O.gemm_dequant(X, codes, S, Z, q, G))
        # element by element (the largest result of a row of eight columns can be small): a weight is rounded to eleven
        # bits (2^-12 of it); twice that leaves room for subnormal weights and the fp32 sums
        bounds.append(2.0 ** -11 * np.abs(X.astype(np.float64)) @ np.abs(O.dequantize(codes, S, Z, q, G)))
    batch = B.GemmBatch(descs, packs, Xs, Ys, out_f32=True)
    for _ in range(2):
        batch.launch()
        for Y, ref, bound in zip(Ys, refs, bounds):
            assert (np.abs(Y.cpu().numpy().astype(np.float64) - ref) <= bound).all()


@pytest.mark.parametrize("K,N,M", [(256, 65536, 24), (1024, 65536, 16)])
def test_wide_and_short_launches_are_not_left_to_it(K, N, M):
    """Many workgroups of few chunks each pay its start and end per round: 2.7 and 1.5 times the tiled kernel's time, to which
    they go (1.0 measured)."""
    desc, packed = pack_on_gpu(*synth.make_weight(K, N, 1, 64, "short-wide"), 1, 64)
    x, ws = dev(synth.make_x(M, K, "short-wide")), B.alloc_workspace(desc, M)
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")

    def us(path):
        B.set_gemm_path(path)
        try:
            best = 1e9
            for _ in range(5):
                B.hlq_lut_gemm(desc, packed, x, y, ws=ws)
                a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(50):
                    B.hlq_lut_gemm(desc, packed, x, y, ws=ws)
                e.record()
                e.synchronize()
                best = min(best, a.elapsed_time(e) * 20)
            return best
        finally:
            B.set_gemm_path(B.GEMM_AUTO)

    assert us(B.GEMM_AUTO) < 1.25 * us(B.GEMM_MFMA_FP16)
