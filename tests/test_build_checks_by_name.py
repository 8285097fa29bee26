"""The build-time check of a kernel that names its accumulators in asm (csrc/check_mfma_hazards.py --by-name): AGPRs as the
compiler prints an asm statement's operands, and none outside such statements; and the listings that the build checks are of the
code that it links."""
import os
import sys

import pytest

from test_build_checks import chk


def test_registers_as_asm_operands_print_them():
    assert chk.aregs("a[108], v[0:3], a[0x6c:0x6f]") == {108, 109, 110, 111}
    assert chk.aregs("a[4:7], a5, s[0:3]") == {4, 5, 6, 7}


@pytest.mark.parametrize("line,found", [("v_accvgpr_write_b32 a3, 0", 1), ("buffer_store_dwordx4 a[8:11], v1, s[0:3], 0 offen", 1),
                                        ("v_add_u32_e32 v0, s1, v2", 0), (".set x.num_agpr, 128", 0)])
def test_accumulators_outside_asm_statements(line, found):
    body = "\t;;#ASMSTART\n\tv_accvgpr_read_b32 v1, a[0x40]\n\t;;#ASMEND\n\t%s\n" % line
    assert len(chk.compiler_placed(body.split("\n"))) == found


def test_named_accumulators_keep_their_distance():
    mfma = "\tv_mfma_f32_16x16x32_bf16 a[0x6c:0x6f], v[0:3], v[4:7], a[0x6c:0x6f]"
    read = "\tv_accvgpr_read_b32 v9, a[0x6d]\n"
    assert chk.check_kernel("k", (mfma + "\n" + read).split("\n"))[1]
    assert not chk.check_kernel("k", (mfma + "\n\ts_nop 15\n\ts_nop 15\n" + read).split("\n"))[1]


def test_listings_are_compiled_like_the_objects(monkeypatch):
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import __graft_entry__ as entry
    ran = []
    monkeypatch.setattr(entry, "_run", ran.append)
    for src in ("kernels_gemm.hip", "kernels_gemm_pp.hip"):
        monkeypatch.setitem(entry.EXTRA_FLAGS, src, ["-DOF_" + src[:-4]])
    entry.build()                       # every command goes to `ran` instead

    def flags(cmd, how):
        src = [a for a in cmd if a.endswith(".hip")][0]
        return os.path.basename(src), [a for a in cmd if a not in how + [src, cmd[cmd.index("-o") + 1]]]

    objects = dict(flags(c, ["-c"]) for c in ran if "-c" in c and any(a.endswith(".hip") for a in c))
    listings = dict(flags(c, ["-S", "--cuda-device-only"]) for c in ran if "-S" in c)
    assert sorted(listings) == ["kernels_gemm.hip", "kernels_gemm_pp.hip"]
    for src, f in listings.items():
        assert f == objects[src] and "-DOF_" + src[:-4] in f
