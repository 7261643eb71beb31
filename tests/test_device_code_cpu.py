"""What must hold in the built gfx950 code itself, read from the library's disassembly (no GPU)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2406_17145_amd import binding as B

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm/bin/llvm-objdump")


COPY = re.compile(r"buffer_load_dwordx4 v\d+, s\[(\d+):(\d+)\], 0 offen lds")


def _code_objects(tmp_path):
    """Disassembly of every gfx950 code object bundled into the library."""
    if not os.path.exists(B.LIB_PATH):
        from paper_2406_17145_amd.build import build_library
        build_library(verbose=False)
    data, magic, at = open(B.LIB_PATH, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        entry = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(magic))[0]):
            off, size, name = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + name]:
                obj = tmp_path / "object"
                obj.write_bytes(data[at + off:at + off + size])
                yield subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
            entry += 24 + name
        at += len(magic)


def _instructions(text):
    """[(instruction, indices of those that can run before it)] in the order of the listing."""
    rows = [re.match(r"\t(.*?)\s*// ([0-9A-F]+): ([0-9A-F]+)", line) for line in text.splitlines()]
    rows = [(m[1], int(m[2], 16), int(m[3], 16)) for m in rows if m]
    at = {addr: i for i, (_, addr, _) in enumerate(rows)}
    before = [[] for _ in rows]
    for i, (ins, addr, word) in enumerate(rows):
        if ins.startswith(("s_branch", "s_cbranch")):
            off = word & 0xffff
            before[at[addr + 4 + 4 * (off - 0x10000 if off & 0x8000 else off)]].append(i)
        if i + 1 < len(rows) and not ins.startswith(("s_branch", "s_endpgm", "s_setpc")):
            before[i + 1].append(i)
    return [(ins, b) for (ins, _, _), b in zip(rows, before)]


def _too_early(code):
    """(copies into LDS, those that on some path follow a vector write of their descriptor by less than five wait states)."""
    copies, early = 0, []
    for i, (line, _) in enumerate(code):
        m = COPY.match(line)
        if not m:
            continue
        copies += 1
        regs, todo, seen = range(int(m[1]), int(m[2]) + 1), [(j, 0) for j in code[i][1]], set()
        while todo:
            j, waited = todo.pop()
            if waited >= 5 or (j, waited) in seen:
                continue
            seen.add((j, waited))
            ins = code[j][0]
            w = re.match(r"v_\S+ s(?:(\d+)|\[(\d+):(\d+)\])|v_\S+ v\S+, s\[(\d+):(\d+)\], \S+, \S+", ins)
            if w and any(int(w[1] or w[2] or w[4]) <= r <= int(w[1] or w[3] or w[5]) for r in regs):
                early.append((i, ins))
                continue
            nop = re.fullmatch(r"s_nop (\d+)", ins)
            todo += [(k, waited + (int(nop[1]) + 1 if nop else 1)) for k in code[j][1]]
    return copies, early


def test_the_check_finds_a_copy_that_comes_too_early():
    listing = """
\tv_readfirstlane_b32 s{}, v1                                // 000000000100: 7E0A0501
\ts_mov_b32 m0, s9                                           // 000000000104: BEFC0009
\ts_nop {}                                                    // 000000000108: BF800000
\tbuffer_load_dwordx4 v2, s[4:7], 0 offen lds                // 00000000010C: E0DD1000 80010002
\tv_readlane_b32 s{}, v9, 3                                  // 000000000114: D2890006 00010709
\ts_cbranch_scc1 65529                                       // 00000000011C: BF85FFF9
\ts_endpgm                                                   // 000000000120: BF810000
"""
    def early(*numbers):
        return _too_early(_instructions(listing.format(*numbers)))
    assert early(5, 2, 8) == (1, [(3, "v_readfirstlane_b32 s5, v1")]) and early(5, 3, 8) == (1, [])
    assert early(8, 1, 6) == (1, [(3, "v_readlane_b32 s6, v9, 3")]) and early(8, 2, 6) == (1, [])       # (around the loop)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs the toolchain's disassembler")
def test_copies_into_lds_wait_for_their_descriptor(tmp_path):
    """A memory instruction may read a scalar register that a vector instruction has written five wait states later at the earliest.
    The copies are written out, so the compiler does not see to it."""
    copies = 0
    for text in _code_objects(tmp_path):
        n, early = _too_early(_instructions(text))
        copies += n
        assert not early, early[:4]
    assert copies >= 100
