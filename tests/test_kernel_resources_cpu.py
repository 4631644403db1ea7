"""What the compiler made of the kernels, from the code-object metadata inside
the built library: no GPU needed."""
import struct

import msgpack

import paper_2405_18628_amd as ppd


def _kernels():
    """The metadata of every kernel in the library (AMDGPU ELF images carry it as
    a msgpack note)."""
    blob = open(ppd.LIB_PATH, "rb").read()
    out, at = [], blob.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:  # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", blob, at + 40)
            size, n = struct.unpack_from("<HH", blob, at + 58)
            for i in range(n):
                h = at + shoff + i * size
                kind, = struct.unpack_from("<I", blob, h + 4)
                off, length = struct.unpack_from("<QQ", blob, h + 24)
                if kind != 7:  # SHT_NOTE
                    continue
                nsz, dsz, ntype = struct.unpack_from("<III", blob, at + off)
                if blob[at + off + 12:at + off + 12 + 6] == b"AMDGPU" and ntype == 32:
                    d = at + off + 12 + (nsz + 3) // 4 * 4
                    out += msgpack.unpackb(blob[d:d + dsz])["amdhsa.kernels"]
        at = blob.find(b"\x7fELF", at + 4)
    return out


def test_matrix_kernels_spill_no_registers():
    """Registers that do not fit go to scratch memory, a round trip in the middle
    of loops whose loads are counted: every tile is sized so that none do."""
    kernels = [k for k in _kernels() if any(n in k[".name"] for n in ("gemm", "attn", "attention"))]
    names = [k[".name"] for k in kernels]
    assert sum("gemm_bf16_kernel" in n for n in names) > 100 and any("attn_bf16_kernel" in n for n in names)
    spilled = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels if k[".private_segment_fixed_size"]}
    assert not spilled, spilled
