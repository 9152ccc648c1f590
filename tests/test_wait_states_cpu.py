"""The wait states that gfx950 leaves to the program, checked in the built library's own device code: a vector memory
instruction reads a scalar register no earlier than five wait states after a VALU instruction wrote it, and a load into
LDS follows the write of m0 by at least one.  The compiler sees to both except inside inline assembly."""
import os
import re
import struct
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def device_code(lib):
    """The gfx950 code objects bundled in lib."""
    data = open(lib, "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name] and size:
                yield data[at + off:at + off + size]
            p += 24 + name
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def scalars(text):
    out = set()
    for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        lo, hi = (m[1], m[2]) if m[1] else (m[3], m[3])
        out.update(range(int(lo), int(hi) + 1))
    if re.search(r"\bvcc\b", text):
        out.add("vcc")
    return out


def short_waits(listing):
    """(wait states to the nearest VALU write of a scalar that a vector memory instruction reads, or to the write of m0
    before a load into LDS; the instruction) of every such instruction that follows too soon."""
    found, loads = [], 0
    recent = []   # (wait states since, scalars written by VALU, writes m0), the last few instructions
    for line in listing.splitlines():
        ins = line.split("//")[0].strip()
        if not ins or ins.endswith(":") or ins.startswith("/"):
            continue
        op, _, args = ins.partition(" ")
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            reads = scalars(args)
            to_lds = "_lds_" in op or args.split()[-1:] == ["lds"]
            loads += to_lds
            for since, written, m0 in recent:
                if (since < 5 and written & reads) or (to_lds and m0 and since < 1):
                    found.append((since, ins))
        states = int(args, 0) + 1 if op == "s_nop" else 1
        recent = [(s + states, w, m) for s, w, m in recent if s + states < 5]
        dst = ",".join(args.split(",")[:2 if "_co_" in op or "div_scale" in op else 1])
        recent.append((0, scalars(dst) if op.startswith("v_") else set(), op.startswith("s_") and dst == "m0"))
    return found, loads


def test_rule_sees_a_short_wait():
    near = "v_readfirstlane_b32 s5, v3\ns_mov_b32 m0, s7\ns_nop {}\nglobal_load_lds_dwordx4 v4, s[4:5]"
    assert short_waits(near.format(0)) == ([(2, "global_load_lds_dwordx4 v4, s[4:5]")], 1)
    assert short_waits(near.format(2))[0] and not short_waits(near.format(3))[0]
    assert short_waits("s_mov_b32 m0, s7\nglobal_load_lds_dword v4, s[4:5]")[0]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_device_code_keeps_its_wait_states(tmp_path):
    import paper_1707_00516_amd as fid
    loads = 0
    for i, code in enumerate(device_code(fid.LIB_PATH)):
        path = tmp_path / f"code{i}.elf"
        path.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                                 capture_output=True, text=True, check=True).stdout
        found, n = short_waits(listing)
        loads += n
        assert not found, (len(found), found[:5])
    assert loads > 0
