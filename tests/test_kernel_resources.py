"""What the compiler made of the kernels, from the library's own code objects.

Private memory: the kernels of the call that allocates no device memory must not
need any, since the runtime would have to find it at the launch.

Copies ahead of a join: where lanes that left a divergent loop or branch join
again, the execution mask is restored by `s_or_b64 exec, exec, ...`.  A copy of a
live register that the compiler puts before that instruction copies the lanes
that came last, or none, and what reads the copy later gets leftover values: the
final lengths of an optimisation once went to such an address."""
import os
import re
import struct
import subprocess

import pytest

import paper_1811_11007_amd as pt

TOOLS = "/opt/rocm/llvm/bin"


def code_objects(tmp_path):
    """Files with the library's code objects."""
    path = os.path.join(os.path.dirname(pt.__file__), "libpt.so")
    data = open(path, "rb").read()
    at = [m.start() for m in re.finditer(b"\x7fELF", data)
          if struct.unpack_from("<H", data, m.start() + 18)[0] == 224]  # e_machine: AMD GPU
    assert at, "no code objects in the library"
    for i, o in enumerate(at):
        f = tmp_path / ("code_object%d" % i)
        f.write_bytes(data[o:at[i + 1] if i + 1 < len(at) else len(data)])
        yield str(f)


def run(tool, *args):
    return subprocess.run([os.path.join(TOOLS, tool), *args], stdout=subprocess.PIPE, text=True, check=True).stdout


def kernels(tmp_path):
    """(name, bytes of private memory per lane) of every kernel in libpt.so."""
    out = []
    for f in code_objects(tmp_path):
        for k in run("llvm-readelf", "--notes", f).split(".agpr_count:")[1:]:
            out.append((re.search(r"\.name:\s+(\S+)", k).group(1),
                        int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1))))
    return out


def copies_before_joins(listing):
    """(kernel, address, copies) wherever a basic block of a disassembly starts
    with copies between vector registers and then restores the execution mask.
    (Where the restoring instruction is itself branched to, the copies before it
    are those of the lanes that did not skip them.)"""
    code, targets, base, kernel = [], set(), {}, ""
    for line in listing.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:$", line)
        if m:
            kernel = m.group(2)
            base[kernel] = int(m.group(1), 16)
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if m:
            code.append((kernel, int(m.group(2), 16), m.group(1)))
            if re.match(r"s_c?branch", m.group(1)):
                to = re.search(r"<([^+>]+)(?:\+0x([0-9a-f]+))?>", line)
                targets.add(base[to.group(1)] + int(to.group(2) or "0", 16))
    copy = re.compile(r"v_accvgpr_(read|write|mov)|v_mov_b(32|64)\S* [va][\d\[:\]]+, [va][\d\[]")
    found = []
    for i, (kernel, addr, _) in enumerate(code):
        if addr not in targets and not (i and re.match(r"s_c?branch", code[i - 1][2])):
            continue
        copies = []
        for k, at, text in code[i:]:
            if k != kernel or (at != addr and at in targets):
                break
            if copy.match(text):
                copies.append(text)
            elif re.match(r"s_or_b64 exec, exec,", text):
                if copies:
                    found.append((kernel, hex(addr), copies))
                break
            elif not re.match(r"s_(waitcnt|nop|mov_b32|movk_i32|add|sub|lshl|mul)", text):
                break
    return found


def test_copies_before_joins_are_found():
    """The sequence that the compiler once made, and the same after the join."""
    text = """
0000000000001000 <kernel>:
\ts_cbranch_execz 7    // 000000001000: BF880007 <kernel+0x14>
\tv_add_f64 v[4:5], v[4:5], v[6:7]    // 000000001004: 00000000
\ts_andn2_b64 exec, exec, s[6:7]    // 00000000100C: 00000000
\ts_cbranch_execnz 65531    // 000000001010: BF89FFFB <kernel+0x4>
\t%s    // 000000001014: 00000000
\t%s    // 00000000101C: 00000000
\ts_barrier    // 000000001020: 00000000
"""
    copy, join = "v_accvgpr_write_b32 a20, v68", "s_or_b64 exec, exec, s[4:5]"
    assert copies_before_joins(text % (copy, join)) == [("kernel", "0x1014", [copy])]
    assert copies_before_joins(text % (join, copy)) == []


@pytest.mark.skipif(not os.path.isdir(TOOLS), reason="no LLVM tools")
def test_no_copies_before_joins(tmp_path):
    pt.lib()
    found = [x for f in code_objects(tmp_path) for x in copies_before_joins(run("llvm-objdump", "-d", f))]
    assert not found, found


@pytest.mark.skipif(not os.path.isdir(TOOLS), reason="no LLVM tools")
def test_likelihood_kernels_need_no_private_memory(tmp_path):
    pt.lib()
    found = [k for k in kernels(tmp_path) if re.search("k_prune|k_pmat_lanes|k_tile_sums", k[0])]
    assert len(found) >= 27, found
    assert not [k for k in found if k[1]], [k for k in found if k[1]]
