"""What the compiler gave the kernels of the built library, from the metadata that it puts beside their
code: registers that fit, no scratch memory (the library allocates no device memory, and scratch
is memory that the runtime would provide for it).  No GPU needed."""
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

import paper_2511_13732_amd as pcg
from paper_2511_13732_amd import build as hip_build

ELF, EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = b"\x7fELF", 224, 7, 32


def kernels(path):
    """The metadata of every kernel in the code objects that the library at `path` holds."""
    blob, found = open(path, "rb").read(), []
    at = blob.find(ELF, 1)
    while at >= 0:
        machine, = struct.unpack_from("<H", blob, at + 18)
        sections, = struct.unpack_from("<Q", blob, at + 40)
        count, = struct.unpack_from("<H", blob, at + 60)
        for i in range(count if machine == EM_AMDGPU else 0):
            _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", blob, at + sections + 64 * i)
            if kind != SHT_NOTE:
                continue
            note = at + off
            while note < at + off + size:
                name_size, desc_size, note_type = struct.unpack_from("<III", blob, note)
                desc = note + 12 + (name_size + 3) // 4 * 4
                if note_type == NT_AMDGPU_METADATA:
                    found += msgpack.unpackb(blob[desc:desc + desc_size])["amdhsa.kernels"]
                note = desc + (desc_size + 3) // 4 * 4
        at = blob.find(ELF, at + 4)
    return found


@pytest.mark.skipif(hip_build.sanitize_requested(), reason="the sanitizer build compiles for another optimisation level")
def test_no_kernel_uses_scratch():
    found = kernels(pcg.lib_path())
    names = {k[".name"] for k in found}
    for part in ("row_stats_kernel", "accept_delta_kernel", "gather_kernel", "gather_prepared_kernel", "finalize_kernel",
                 "finalize_sums_kernel", "small_step_kernel", "accept_thin_kernel", "propose_row_kernel", "propose_kernel",
                 "row_weights_kernel", "weights_parts_kernel", "weights_kernel", "asg_normalize_kernel",
                 "asg_similarity_kernel", "asg_refine_kernel", "asg_sort_kernel", "asg_compact_kernel"):
        # as a whole name: mangled, its length stands in front of it
        assert any(f"{len(part)}{part}" in n for n in names), part
    bad = [(k[".name"], k[".vgpr_count"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in found
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"] or k.get(".uses_dynamic_stack")]
    assert not bad, f"{len(bad)} of {len(found)} kernels: {bad[:3]}"
    # a workgroup finds room for its registers: 512 a lane on each of the four SIMDs, in steps of 8
    for k in found:
        waves = (k[".max_flat_workgroup_size"] + 255) // 256
        assert (k[".vgpr_count"] + 7) // 8 * 8 * waves <= 512, k[".name"]
        assert k[".group_segment_fixed_size"] <= 160 * 1024, k[".name"]
