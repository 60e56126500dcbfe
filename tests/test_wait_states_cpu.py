"""The built device code keeps the target's wait states between a vector
instruction that writes a scalar register and a memory instruction that reads it.

On gfx9 and CDNA a VMEM instruction may read an SGPR that a VALU instruction
(v_readfirstlane, a compare, a carry) wrote only five wait states later, and the
hardware does not interlock it.  The compiler keeps the distance between its own
instructions but not for loads inside inline assembly, so every memory instruction
of the library is checked here on the disassembly, along every path that leads to
it.  The last test plants short distances in a listing."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2609_24089_amd as fb
from paper_2609_24089_amd.build import hipcc

WAIT_STATES = 5


def llvm_tool(name):
    return os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc()))), "llvm", "bin", name)


def code_objects(tmp):
    """The library's gfx950 code objects, extracted into `tmp`."""
    if not os.path.exists(fb.LIB_PATH):
        from paper_2609_24089_amd.build import build_library
        build_library()
    lib = os.path.join(tmp, "lib.so")
    shutil.copy(fb.LIB_PATH, lib)
    subprocess.run([llvm_tool("llvm-objdump"), "--offloading", lib], check=True, capture_output=True, cwd=tmp)
    objs = sorted(os.path.join(tmp, n) for n in os.listdir(tmp) if n.endswith("gfx950"))
    assert objs
    return objs


def disassembly(obj):
    return subprocess.run([llvm_tool("llvm-objdump"), "-d", "--no-show-raw-insn", obj], check=True,
                          capture_output=True, text=True).stdout


LINE = re.compile(r"^\s+([a-z]\w+)(?: (.*?))?\s*// ([0-9A-F]+):(?: [0-9A-F]{8})*(?: <(.+)\+0x([0-9a-f]+)>| <(.+)>)?")
SREG = re.compile(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]|\b(vcc)\b")
# vector instructions whose scalar result is their second operand
SECOND = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_mad_[iu]64|v_div_scale")


def sregs(text):
    out = set()
    for one, lo, hi, vcc in SREG.findall(text):
        if vcc:
            out.add("vcc")
        elif one:
            out.add(int(one))
        else:
            out.update(range(int(lo), int(hi) + 1))
    return out


def valu_writes(op, args):
    """Scalar registers that a vector instruction writes."""
    operands = re.split(r",\s*", args)
    if SECOND.match(op):
        return sregs(operands[1])
    if op.startswith(("v_cmp", "v_readfirstlane", "v_readlane")):
        return sregs(operands[0])
    return set()


def short_distances(listing):
    """(address, instruction, register) of every memory instruction of a listing
    that reads a scalar register fewer than WAIT_STATES after a vector write."""
    code = []  # (op, args, address, branch target)
    start = {}
    for line in listing.splitlines():
        sym = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if sym:
            start[sym.group(2)] = int(sym.group(1), 16)
            continue
        m = LINE.match(line)
        if m:
            op, args, addr, base, off, exact = m.groups()
            target = None
            if op in ("s_branch",) or op.startswith("s_cbranch"):
                target = (exact, 0) if exact else (base, int(off, 16)) if base else None
                assert target is not None, line
            code.append((op, args or "", int(addr, 16), target))
    at = {c[2]: i for i, c in enumerate(code)}
    jumps = {}
    for i, c in enumerate(code):
        if c[3] is not None:
            jumps.setdefault(at[start[c[3][0]] + c[3][1]], []).append(i)
    found = []
    for i, (op, args, addr, _) in enumerate(code):
        if not op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            continue
        reads = sregs(args)
        if not reads:
            continue
        todo, seen = [(i, 0)], set()
        while todo:  # backwards over every path, as far as the wait states reach
            j, states = todo.pop()
            before = list(jumps.get(j, []))
            if j > 0 and code[j - 1][0] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                before.append(j - 1)
            for b in before:
                o, a = code[b][0], code[b][1]
                hit = reads & valu_writes(o, a) if o.startswith("v_") else set()
                if hit:
                    found.append((hex(addr), f"{op} {args}", sorted(map(str, hit)), states))
                n = states + (int(a, 0) + 1 if o == "s_nop" else 1)
                if n < WAIT_STATES and (b, n) not in seen:
                    seen.add((b, n))
                    todo.append((b, n))
    return found, sum(c[0].startswith("buffer_load") and c[1].endswith("lds") for c in code)


def test_memory_instructions_keep_the_wait_states(tmp_path):
    found, copies = [], 0
    for obj in code_objects(str(tmp_path)):
        bad, n = short_distances(disassembly(obj))
        found += [(os.path.basename(obj), *b) for b in bad]
        copies += n
    assert copies > 100  # the tile copies were seen
    assert not found, (len(found), found[:5])


@pytest.mark.parametrize("nop,bad", [(0, 1), (2, 1), (3, 0), (4, 0)])
def test_the_check_sees_a_short_distance(nop, bad):
    text = f"""
0000000000001000 <kernel>:
	v_readfirstlane_b32 s40, v40                               // 000000001000:
	s_mov_b32 m0, s6                                           // 000000001004:
	s_nop {nop}                                                // 000000001008:
	buffer_load_dwordx4 v117, s[40:43], 0 offen lds            // 00000000100C:
	s_cbranch_scc1 65530                                       // 000000001014: <kernel+0x4>
	s_endpgm                                                   // 000000001018:
"""
    assert len(short_distances(text)[0]) == bad
