"""The library's kernels, disassembled: a vector-memory instruction that takes its address from scalar registers comes at least five wait
states after a vector instruction has written one of them (v_readfirstlane, v_readlane, comparisons).  The hardware does not wait, and
the compiler does not look into inline assembly: the loads that write LDS bring their own wait states (lds_load_device.h)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_17469_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
SCALAR = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b|\b(vcc)\b")
TWO_RESULTS = re.compile(r"v_(add|addc|sub|subb|subrev|subbrev)_co_|v_mad_[ui]64|v_div_scale")
VCC = (106, 107)


def scalars(text):
    out = set()
    for lo, hi, one, vcc in SCALAR.findall(text):
        out.update(range(int(lo), int(hi) + 1) if lo else VCC if vcc else (int(one),))
    return out


def too_early(lines, need=5):
    """(lines, how many wait states there were) of loads and stores that come too early; `lines`: a kernel in the order of its code."""
    found, since = [], {}
    for line in lines:
        op, _, rest = line.partition(" ")
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            found += [(line, since[r]) for r in scalars(rest) if since.get(r, need) < need]
        states = int(rest, 0) + 1 if op == "s_nop" else 1
        since = {r: n + states for r, n in since.items() if n + states < need}
        results = rest.split(",")
        if op.startswith("v_"):
            for r in scalars(" ".join(results[:2] if TWO_RESULTS.match(op) else results[:1])):
                since[r] = 0
        elif op.startswith("s_"):                        # (the hardware waits for a scalar instruction's result)
            for r in scalars(results[0]):
                since.pop(r, None)
    return found


def test_the_count():
    load = "global_load_lds_dwordx4 v1, s[4:5]"
    early = ["v_readfirstlane_b32 s5, v2", "s_mov_b32 s0, m0", "s_mov_b32 m0, s3", "s_nop 0", load]
    assert too_early(early) == [(load, 3)]
    assert too_early(early[:3] + ["s_nop 2", load]) == []
    assert too_early(["v_readlane_b32 s4, v2, 1", "s_mov_b64 s[4:5], s[6:7]", load]) == []
    assert len(too_early(["v_add_co_u32_e64 v0, s[4:5], v1, v2", load])) == 2


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_scalar_addresses_are_not_read_too_early(tmp_path):
    shutil.copy(binding.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    objects = sorted(glob.glob(str(tmp_path / "*gfx950")))
    assert objects
    found, loads = {}, 0
    for o in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", o], check=True, capture_output=True, text=True).stdout
        kernel, lines = None, []
        for line in text.splitlines() + ["0000 <end>:"]:
            if line.endswith(">:"):
                bad = too_early(lines)
                if bad:
                    found[kernel] = bad[:3]
                kernel, lines = line.split("<")[-1][:-2], []
            else:
                line = line.split("//")[0].strip()
                if line:
                    lines.append(line)
                    loads += line.startswith("global_load_lds") and not line.endswith("off")
    assert loads > 100                                   # (that the loads in question are among what was read)
    assert not found, (len(found), dict(list(found.items())[:3]))
