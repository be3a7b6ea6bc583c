"""The D = 64 dK/dV kernels keep their scalars in scalar registers: spilled ones live in lanes of vector registers, and every tile of the loop fetches
them from there (32:4 heads x 1200 tokens, the whole backward pass, 65 us with 91 of them spilled, 57 without).  Read from the code objects' notes in
the library built here.  The pinned loops of D = 128 (attn_fwd_pinned at 250 of the 256 registers that let two blocks share a unit, dK/dV) keep everything in registers,
too: their instructions have their places, and scratch accesses would stand among them.  No GPU needed."""
import struct

import msgpack

from paper_2411_15871_amd import dhelix as dh


def kernel_notes():
    """.name -> metadata of every kernel in the library (AMDGPU notes: name "AMDGPU", type 32, a msgpack map)."""
    blob, out, at = open(dh._LIB_PATH, "rb").read(), {}, 0
    while True:
        at = blob.find(b"AMDGPU\0\0", at)
        if at < 0:
            return out
        namesz, size, kind = struct.unpack_from("<III", blob, at - 12)
        if namesz == 7 and kind == 32:
            for k in msgpack.unpackb(blob[at + 8: at + 8 + size])["amdhsa.kernels"]:
                out[k[".name"]] = k
        at += 8


def test_attention_backward_spills_no_scalars():
    notes = kernel_notes()
    backward = {n: k for n, k in notes.items() if "attn_bwd_bf16_kernel" in n or "attn_bwd_dkv_bf16_kernel" in n}
    assert len(backward) == 4  # both head widths, dK/dV alone and beside dQ
    for name, k in backward.items():
        assert k[".sgpr_spill_count"] == 0 and k[".vgpr_spill_count"] == 0, name


def test_pipelined_forward_stays_in_registers():
    forward = {n: k for n, k in kernel_notes().items() if "attn_fwd_pinned_bf16_kernel" in n or "attn_fwd_bf16_kernel" in n}
    assert len(forward) == 3  # the pipelined loop, and the loop in phases at both head widths
    for name, k in forward.items():
        assert k[".vgpr_count"] <= 256, name
        assert k[".sgpr_spill_count"] == 0 and k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name
