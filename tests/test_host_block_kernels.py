"""The row-owning block kernels as they were built: their register budgets are full (a tile's weights, accumulators and fragments in
flight), and a register more is a spill, whose reload waits for every weight that is on its way."""
import struct

import pytest
from paper_2404_13528_amd import binding as sm

NOTE_TYPE = 32      # metadata of a code object: msgpack under the owner "AMDGPU"


msgpack = pytest.importorskip("msgpack")


def kernels_of(path):
    """{symbol: metadata} of every kernel in the library's code objects."""
    sm.lib()
    with open(path, "rb") as f:
        data = f.read()
    out, at = {}, data.find(b"AMDGPU\0\0")
    while at >= 0:
        owner, size, kind = struct.unpack_from("<III", data, at - 12)
        if (owner, kind) == (7, NOTE_TYPE):
            out.update((k[".name"], k) for k in msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"])
        at = data.find(b"AMDGPU\0\0", at + 8)
    return out


def test_no_spills():
    block = {n: k for n, k in kernels_of(sm.LIB_PATH).items() if "mlp_fused_kernel" in n or "mlp64" in n}
    assert len(block) == 27, sorted(block)      # widths, projection or not, second output
    assert not {n: k[".vgpr_spill_count"] for n, k in block.items() if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
