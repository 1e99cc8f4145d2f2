"""Conditional scalar branches of the kernels as the compiler wrote them.

The compiler has been seen to lose the compare of a wave-uniform branch: in a
loop whose uniform values it kept in vector registers it placed the merge of
another condition (s_andn2_b64, s_and_b64, s_or_b64) between the compare and
the branch, all of which set the condition bit, and then dropped the compare as
unused.  The branch went by the merge's result, the walk entered cells that no
target had opened, and read out of bounds.  The source was right, so only the
compiled code shows it."""
from __future__ import annotations

import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_1005_5312_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# 64-bit logic (lane masks); each sets the condition bit from its own result
MASK_LOGIC = re.compile(r"s_(and|andn2|or|orn2|xor|nand|nor|xnor|not)_b64$")
# scalar instructions that leave the condition bit alone
KEEPS = re.compile(r"s_(mov|movk|cmov|cselect|load|buffer|store|waitcnt|nop|branch|cbranch|mul|mulk|getpc|setpc|swappc|"
                   r"endpgm|barrier|sleep|setprio|ff0|ff1|flbit|sext|brev|bitset|bfm|pack|sendmsg|getreg|setreg|"
                   r"memtime|memrealtime|dcache|icache|inst_prefetch)")


def lost_compares(listing):
    """(kernel, line) of every s_cbranch_scc whose condition bit was last set by
    lane-mask logic."""
    kernel, setter, found = "", "", []
    for number, line in enumerate(listing.splitlines(), 1):
        code = line.split(";")[0].strip()
        if code.endswith(":"):
            kernel = code[:-1] if code.startswith("_Z") else kernel
            setter = ""
            continue
        op = code.split()[0] if code else ""
        if op.startswith("s_cbranch_scc"):
            if MASK_LOGIC.match(setter):
                found.append((kernel, number))
        elif op.startswith("s_") and not KEEPS.match(op):
            setter = op
    return found


def test_finds_a_lost_compare():
    listing = """
_Z4walk:
.LBB15_31:                              ;   in Loop
	v_cmp_lt_i32_e32 vcc, 1, v31
	s_andn2_b64 s[0:1], s[18:19], exec
	s_and_b64 s[18:19], vcc, exec
	s_or_b64 s[18:19], s[0:1], s[18:19]
	s_cbranch_scc1 .LBB15_35
"""
    assert lost_compares(listing) == [("_Z4walk", 8)]
    assert lost_compares(listing.replace("	s_cbranch", "	s_cmp_eq_u64 s[2:3], 0\n	s_cbranch")) == []


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_every_branch_has_its_compare(tmp_path):
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")] + ["--cuda-device-only", "-S", "-w"]

    def listing(src):
        out = tmp_path / (os.path.basename(src) + ".s")
        subprocess.run([HIPCC, *flags, "-I", os.path.join(B.ROOT, "include"), "-o", str(out), src], check=True,
                       capture_output=True)
        return out.read_text()

    with ThreadPoolExecutor(4) as pool:
        listings = list(pool.map(listing, B.sources()))
    branches = sum(t.count("s_cbranch_scc") for t in listings)
    assert branches > 100, branches
    for src, text in zip(B.sources(), listings):
        assert lost_compares(text) == [], os.path.basename(src)
