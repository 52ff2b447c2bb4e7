"""HLQ_GEMV_W and HLQ_GEMV_CPW (read once per process) force the launch shape as hlq_set_gemv_plan does, on launches of
either one-row kernel; a knob that is set wins over them.  Host arithmetic only."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
QUERY = """
from paper_2510_19482_amd import binding as B
for K, N, q, G in ((4096, 1024, 2, 128), (14336, 4096, 2, 128), (4096, 28672, 2, 32)):
    for W, cpw in ((0, 0), (4, 3)):
        B.set_gemv_plan(0, W, cpw)
        try:
            i = B.gemv_plan_query([B.make_desc(K, N, q, G)], 1)[0]
            print(i.waves_per_workgroup, i.waves_per_tile, i.chunks_per_slice, i.slices, i.tile_groups)
        except B.HlqError as e:
            print(e.status)
"""


def plans(**env):
    out = subprocess.run([sys.executable, "-c", QUERY], cwd=ROOT, env=dict(os.environ, **env), capture_output=True, text=True, check=True)
    return [tuple(int(v) for v in line.split()) for line in out.stdout.splitlines()]


def knobs(W, cpw):
    from paper_2510_19482_amd import binding as B
    try:
        B.set_gemv_plan(0, W, cpw)
        infos = [B.gemv_plan_query([B.make_desc(K, N, q, G)], 1)[0] for K, N, q, G in ((4096, 1024, 2, 128), (14336, 4096, 2, 128), (4096, 28672, 2, 32))]
        return [(i.waves_per_workgroup, i.waves_per_tile, i.chunks_per_slice, i.slices, i.tile_groups) for i in infos]
    finally:
        B.set_gemv_plan(0, 0, 0)


@pytest.mark.parametrize("W,cpw", [(2, 0), (0, 5), (16, 2)])
def test_environment_is_the_knob(W, cpw):
    got = plans(**({"HLQ_GEMV_W": str(W)} if W else {}), **({"HLQ_GEMV_CPW": str(cpw)} if cpw else {}))
    assert got[0::2] == knobs(W, cpw) != knobs(0, 0)
    assert got[1::2] == knobs(4, 3)          # the knob wins


def test_values_out_of_range_are_refused():
    assert plans(HLQ_GEMV_W="-3")[0::2] == [(3,)] * 3


@pytest.mark.parametrize("M", [2, 4])
def test_several_rows_do_not_look_at_it(M):
    query = QUERY.replace("], 1)[0]", f"], {M})[0]")
    out = [subprocess.run([sys.executable, "-c", query], cwd=ROOT, env=dict(os.environ, **env), capture_output=True, text=True, check=True).stdout
           for env in ({}, {"HLQ_GEMV_W": "2", "HLQ_GEMV_CPW": "5"}, {"HLQ_GEMV_W": "-3", "HLQ_GEMV_CPW": "-1"})]
    assert out[0] == out[1] == out[2]
