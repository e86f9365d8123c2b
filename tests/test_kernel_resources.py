"""What the fp32 heads' plan counts on, read from the metadata of the built kernels: how many of a kernel's workgroups the registers
and the LDS of a compute unit hold at once.  A kernel that outgrows it runs a launch in more rounds than the plan takes it to."""
import os
import re
import struct

import msgpack
import pytest

from paper_2507_02659_amd import build

# workgroups at once per compute unit by (kernel, row tiles), as f32_plan has them
AT_ONCE = {("lmhead_f32_kernel", 1): 2, ("lmhead_f32_kernel", 2): 4, ("lmhead_f32_kernel", 3): 3,
           ("lmhead_f32_thirds_kernel", 2): 3, ("lmhead_f32_thirds_kernel", 3): 2, ("lmhead_f32_thirds_kernel", 4): 2}
REGISTERS, LDS_BYTES, SIMDS = 512, 160 << 10, 4      # per SIMD and lane, per compute unit


def _kernels():
    """Metadata of the kernels in the built library: its gfx950 code objects are ELF files that hold it as a note."""
    blob = open(build.LIB_PATH, "rb").read()
    for at in (m.start() for m in re.finditer(b"\x7fELF\x02\x01", blob)):
        if struct.unpack_from("<H", blob, at + 18)[0] != 224:            # EM_AMDGPU
            continue
        sections, = struct.unpack_from("<Q", blob, at + 40)
        size, n = struct.unpack_from("<HH", blob, at + 58)
        for i in range(n):
            kind, = struct.unpack_from("<I", blob, at + sections + i * size + 4)
            if kind != 7:                                                # SHT_NOTE
                continue
            note = at + struct.unpack_from("<Q", blob, at + sections + i * size + 24)[0]
            name_size, desc_size, _ = struct.unpack_from("<III", blob, note)
            desc = note + 12 + (name_size + 3) // 4 * 4
            yield from msgpack.unpackb(blob[desc:desc + desc_size], raw=False)["amdhsa.kernels"]


pytestmark = pytest.mark.skipif(not os.path.exists(build.LIB_PATH), reason="not built")


def test_draws_of_eight_wavefronts_are_those_of_many_sequences():
    """The plan takes workgroups of eight wavefronts for more sequences than a launch in front can have hosted: of the kernels that
    test and draw, only the one for that many (the third flag) is built for eight."""
    draws = [k[".name"] for k in _kernels() if re.search(r"\d(accept|final)_draw_kernel", k[".name"]) and k[".max_flat_workgroup_size"] == 512]
    assert draws and all("accept_draw_kernelILi8ELb1ELb1ELb1E" in name for name in draws), draws


def test_draws_without_the_exponentials_are_built_without_their_code():
    """As a runtime choice it cost the draws of one and two turns up to a tenth of the launch, and 112 registers instead of 94."""
    draws = [k for k in _kernels() if "accept_draw_kernelILi8ELb1" in k[".name"] and "ELi16ELb0EEEv" in k[".name"]]
    assert draws
    for k in draws:
        assert k[".vgpr_count"] <= 96, k[".name"]


def test_fp32_heads_fit_a_compute_unit_as_planned():
    seen = set()
    for k in _kernels():
        m = re.search(r"\d(lmhead_f32(?:_thirds)?_kernel)ILi(\d)E", k[".name"])
        if not m:
            continue
        key = (m[1], int(m[2]))
        seen.add(key)
        registers = -(-k[".vgpr_count"] // 8) * 8                        # vector and accumulation registers, allocated by eight
        waves = k[".max_flat_workgroup_size"] // 64
        fit = min(REGISTERS // registers * SIMDS // waves, LDS_BYTES // k[".group_segment_fixed_size"])
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, k[".name"]
        assert fit >= AT_ONCE[key], (k[".name"], registers, fit)
    assert seen == set(AT_ONCE)
