"""Check of the compiled kernels for one fault of the compiler's register allocator.

Where the lanes of a divergent branch meet again, the block has to restore EXEC
(s_or_b64 exec, ...) before anything that is meant for all of them.  With
scalar constants kept over long ranges the allocator (clang 22, ROCm 7.2) forms
some of them anew at the top of such a block, no longer takes the restore for
the block's prologue, and puts the copies of vector registers that it inserts
later in front of it: lanes that did not take the branch are not copied and
read garbage afterwards.  The sources show nothing of it, and results are right
until a lane takes the other side (in FP64, the sine of a huge argument); then
a point's number, and with it the address of its outputs, is garbage.

misplaced() lists every such place in a built library, from the disassembly of
its gfx950 code: a vector or memory instruction between the start of a block
that is entered with lanes missing (the target of s_cbranch_execz, or what
follows s_cbranch_execnz) and the block's EXEC restore.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import re
import struct
import subprocess
import tempfile

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
_SCALAR_RESULT = ("v_readlane", "v_writelane", "v_readfirstlane", "v_cmp", "v_nop")  # not per-lane results
_MEMORY = ("scratch_", "global_", "ds_", "buffer_", "flat_")
_TARGET = re.compile(r"<([^>]+?)(?:\+0x([0-9a-f]+))?>\s*$")


def code_objects(path):
    """The gfx950 code objects in a HIP library's offload bundles."""
    data = open(path, "rb").read()
    at, found = data.find(_MAGIC), []
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(_MAGIC))
        o = at + len(_MAGIC) + 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, o)
            if size and data[o + 24:o + 24 + ln].endswith(b"gfx950"):
                found.append(data[at + off:at + off + size])
            o += 24 + ln
        at = data.find(_MAGIC, at + len(_MAGIC))
    return found


def _find(lines):
    """(block address, instructions before the restore) for one function's disassembly lines."""
    ins, targets = [], set()
    for line in lines:
        text, _, rest = line.partition("//")
        text = text.strip()
        if not text or not rest:
            continue
        op = text.split(None, 1)[0]
        ins.append((int(rest.split(":", 1)[0], 16), op, text))
        if op == "s_cbranch_execz":
            m = _TARGET.search(rest)
            if m:
                targets.add(int(m.group(2) or "0", 16))
    if not ins:
        return []
    base, out, start, pending = ins[0][0], [], None, []
    for addr, op, text in ins:
        if addr - base in targets:
            start, pending = addr - base, []
        if op.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc")):
            start, pending = (addr - base + 4 if op == "s_cbranch_execnz" else None), []
        elif start is None:
            continue
        elif op == "s_or_saveexec_b64" or text.startswith("s_or_b64 exec, exec,"):
            if pending:
                out.append((start, pending))
            start = None
        elif op.startswith("s_") and "exec" in text.split(",", 1)[0]:
            start = None
        elif (op.startswith("v_") and not op.startswith(_SCALAR_RESULT)) or op.startswith(_MEMORY):
            pending.append(text)
    return out


def scan(listing):
    """{function: [(block offset, [instruction, ...]), ...]} for one code object's disassembly text."""
    found, name, lines = {}, None, []
    for line in listing.splitlines() + ["0 <>:"]:
        if line.endswith(">:"):
            bad = _find(lines) if name else []
            if bad:
                found[name] = bad
            name, lines = line[line.index("<") + 1:-2], []
        else:
            lines.append(line)
    return found


def _scan_object(objdump, code):
    with tempfile.NamedTemporaryFile(suffix=".co") as f:
        f.write(code)
        f.flush()
        p = subprocess.run([objdump, "-d", "--no-show-raw-insn", f.name], capture_output=True, text=True)
    if p.returncode:
        raise RuntimeError("disassembly failed: " + p.stderr[-500:])
    return scan(p.stdout)


def misplaced(path, hipcc="/opt/rocm/bin/hipcc", jobs=None):
    """Every misplaced copy in a built library, as scan() gives them."""
    objdump = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    objects = code_objects(path)
    if not objects:
        raise RuntimeError("no gfx950 code in %s" % path)
    found = {}
    with cf.ProcessPoolExecutor(jobs or min(8, os.cpu_count() or 4)) as ex:
        for bad in ex.map(_scan_object, [objdump] * len(objects), objects):
            found.update(bad)
    return found
