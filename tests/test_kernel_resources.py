"""No one-layer kernel of the dense contraction keeps registers in scratch memory: waves that have any start later, at every layer."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")


def kernels(path):
    """name -> metadata of every kernel in the code objects that a library carries (AMDGPU notes, msgpack)."""
    with open(path, "rb") as f:
        data = f.read()
    out = {}
    for m in re.finditer(b"\x7fELF\x02\x01", data):
        base = m.start()
        machine, = struct.unpack_from("<H", data, base + 18)
        if machine != 224:                                   # EM_AMDGPU
            continue
        phoff, = struct.unpack_from("<Q", data, base + 32)
        phentsize, phnum = struct.unpack_from("<HH", data, base + 54)
        for i in range(phnum):
            kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", data, base + phoff + i * phentsize)
            at, end = base + offset, base + offset + size
            while kind == 4 and at + 12 <= end:              # PT_NOTE
                namesz, descsz, ntype = struct.unpack_from("<III", data, at)
                desc = at + 12 + (namesz + 3) // 4 * 4
                if ntype == 32:                              # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(data[desc:desc + descsz])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                at = desc + (descsz + 3) // 4 * 4
    return out


def test_rows_kernels_have_no_scratch():
    from paper_2110_09195_amd import binding
    binding.lib()
    rows = {n: k for n, k in kernels(binding.LIB_PATH).items() if "rows_fp4" in n}
    assert len(rows) >= 15, sorted(rows)
    # (the launch of several layers: two registers, which it is faster with)
    spilled = {n: k[".vgpr_spill_count"] for n, k in rows.items() if k[".vgpr_spill_count"] > (2 if "rows_fp4_many" in n else 0)}
    scratch = {n: k[".private_segment_fixed_size"] for n, k in rows.items() if k[".private_segment_fixed_size"] and "rows_fp4_many" not in n}
    assert not spilled and not scratch, (spilled, scratch)


# Several layers in one launch: outputs past the last-level cache (the instance of template argument true) run faster with two registers in
# scratch memory than in any state without (rows_fp4.hip, PACED), the others with none.
@pytest.mark.parametrize("instance, spilled", [("Lb0", 0), ("Lb1", 2)])
def test_state_of_the_many_layer_kernels(instance, spilled):
    from paper_2110_09195_amd import binding
    binding.lib()
    found = [k[".vgpr_spill_count"] for n, k in kernels(binding.LIB_PATH).items() if "rows_fp4_many" in n and instance in n]
    assert found == [spilled]
