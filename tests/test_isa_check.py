"""The built kernels hold no 64-bit vector shift whose amount is the last
register of the wave's allocation (isa_check.py: the hardware may take it from
v0), and the check sees such a shift where there is one.  CPU only: the small
kernels below are assembled and read, never run."""
import subprocess

import pytest

from paper_2406_13868_amd import _lib, isa_check

KERNEL = """
.amdgcn_target "amdgcn-amd-amdhsa--gfx950"
.text
.globl k
.p2align 8
.type k,@function
k:
  {shift}
  s_endpgm
.rodata
.p2align 6
.amdhsa_kernel k
  .amdhsa_next_free_vgpr {vgprs}
  .amdhsa_next_free_sgpr 16
  .amdhsa_accum_offset {acc}
.end_amdhsa_kernel
.amdgpu_metadata
---
amdhsa.version: [1, 2]
amdhsa.kernels:
  - .agpr_count: {agprs}
    .name: k
    .symbol: k.kd
    .kernarg_segment_size: 0
    .kernarg_segment_align: 4
    .group_segment_fixed_size: 0
    .private_segment_fixed_size: 0
    .wavefront_size: 64
    .sgpr_count: 16
    .vgpr_count: {vgprs}
    .max_flat_workgroup_size: 64
...
.end_amdgpu_metadata
"""


def _needs_tools():
    if not isa_check.have_tools():
        pytest.skip("llvm-objdump not found")


@pytest.mark.parametrize("shift,vgprs,agprs,found", [
    ("v_lshlrev_b64 v[0:1], v7, v[2:3]", 8, 0, True),      # the last of 8
    ("v_lshlrev_b64 v[0:1], v7, v[2:3]", 9, 0, False),     # v8 is allocated
    ("v_lshrrev_b64 v[0:1], v15, v[2:3]", 16, 0, True),
    ("v_ashrrev_i64 v[0:1], v15, v[2:3]", 24, 8, True),    # what follows v15 are accumulation registers
    ("v_lshlrev_b64 v[0:1], v6, v[2:3]", 7, 0, False),     # v7 is part of the allocation
    ("v_lshlrev_b64 v[0:1], s7, v[2:3]", 8, 0, False),     # a scalar amount
    ("v_lshlrev_b32 v0, v7, v2", 8, 0, False),             # a 32-bit shift
])
def test_the_check_sees_a_shift_by_the_last_register(tmp_path, shift, vgprs, agprs, found):
    _needs_tools()
    src, co = tmp_path / "k.s", tmp_path / "k.co"
    src.write_text(KERNEL.format(shift=shift, vgprs=vgprs, agprs=agprs, acc=-(-(vgprs - agprs) // 4) * 4))
    r = subprocess.run([isa_check._tool("clang"), "-x", "assembler", "--target=amdgcn-amd-amdhsa", "-mcpu=gfx950",
                        str(src), "-o", str(co)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    hits = isa_check.shift_hazards(co.read_bytes())
    assert bool(hits) == found and all(h.startswith("k: v_") for h in hits)


def test_the_built_kernels_have_none():
    _needs_tools()
    objects = isa_check.code_objects(_lib.lib()._name)
    assert len(objects) >= 10  # one per kernel source
    isa_check.check(_lib.lib()._name)
