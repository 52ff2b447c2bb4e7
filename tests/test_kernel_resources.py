"""What the compiled kernels take, read from the metadata of the library's own code objects (no GPU needed)."""
import struct

import msgpack
import pytest

from paper_2510_19482_amd import binding as B


def kernels():
    """{symbol: metadata} of every kernel in the library: the AMDGPU metadata note (type 32) of its code objects."""
    blob = open(B.LIB_PATH, "rb").read()
    found, at = {}, 0
    while (at := blob.find(b"AMDGPU\0", at)) >= 0:
        name_size, size, kind = struct.unpack_from("<III", blob, at - 12)
        if (name_size, kind) == (7, 32):
            for k in msgpack.unpackb(blob[at + 8:at + 8 + size]).get("amdhsa.kernels", []):
                found[k[".name"]] = k
        at += 7
    return found


@pytest.mark.parametrize("part", ["hlq_quantize_kernel", "hlq_gemm_mfma_group_reduce_kernel", "hlq_gemm_safe_kernel", "hlq_gemv_cols_kernel",
                                  "hlq_rows_split_kernel", "hlq_gemm_rows_kernel", "hlq_gemm_short_kernel"])
def test_no_scratch_memory(part):
    # scratch is memory that the runtime sets aside per wavefront, and a spilled register is a trip to it in the inner loop
    mine = {n: k for n, k in kernels().items() if part in n}
    assert mine
    assert {n: k[".private_segment_fixed_size"] for n, k in mine.items() if k[".private_segment_fixed_size"]} == {}
