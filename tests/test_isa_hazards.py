"""Two rules that the gfx950 code of every kernel in the built library keeps, whatever the
compiler makes of it:
  * every barrier comes after a wait for the wave's own LDS accesses on every path;
  * the data registers of a store of more than 64 bits are not written by a vector
    instruction within the next two wait states, which the compiler keeps by itself only
    for stores without a register as uniform offset: the store may have read only a part
    of them by then."""
import concurrent.futures as cf
import os
import re
import struct
import subprocess

import pytest

from paper_2205_02380_amd import chasm
from tests.test_lds_waits import LLVM, functions, unwaited_barriers

needs_lib = pytest.mark.skipif(not os.path.exists(chasm.LIB_PATH) or not os.path.exists(f"{LLVM}/llvm-objdump"),
                               reason="no built library or no disassembler")
STORE = re.compile(r"(buffer|global|flat|scratch)_(store|atomic)")
REG = re.compile(r"(?<![a-z_0-9])([va])(?:(\d+)|\[(\d+):(\d+)\])(?![a-z_0-9])")
STATES = 2


def _regs(m):
    return {(m.group(1), i) for i in range(int(m.group(2) or m.group(3)), int(m.group(2) or m.group(4)) + 1)}


def overwritten_stores(ins):
    """(store, overwriting instruction) pairs of one function, along every path."""
    at = {a: i for i, (a, _, _) in enumerate(ins)}
    bad = []

    def follow(i, states, data, store):
        while states < STATES and i < len(ins):
            _, op, target = ins[i]
            name, _, rest = op.partition(" ")
            if name.startswith("v_") and not name.startswith(("v_cmp", "v_readlane", "v_readfirstlane")):
                m = REG.search(rest)
                if m and _regs(m) & data:
                    bad.append((store, op))
                    return
            if name.startswith(("s_branch", "s_cbranch")) and target in at:
                follow(at[target], states + 1, data, store)
            if name.startswith(("s_branch", "s_endpgm")):
                return
            states += 1 + int(rest, 0) if name == "s_nop" else 1
            i += 1

    for i, (_, op, _) in enumerate(ins):
        if STORE.match(op):
            r = [_regs(m) for m in REG.finditer(op)]
            data = r[0] if op.startswith("buffer") and r else r[1] if len(r) > 1 else set()
            if len(data) > 2:
                follow(i + 1, 0, data, op)
    return bad


def code_objects(lib, tmp):
    """The gfx950 code objects of a shared library, each written to a file."""
    fat = os.path.join(tmp, "fat")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", lib, fat + ".so"], check=True)
    with open(fat, "rb") as fh:
        blob = fh.read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", [], 0
    while (at := blob.find(magic, at)) >= 0:
        p = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, p - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + n]
            p += 24 + n
            if name.endswith(b"gfx950") and size:
                out.append(os.path.join(tmp, f"{len(out)}.co"))
                with open(out[-1], "wb") as fh:
                    fh.write(blob[at + off:at + off + size])
        at += len(magic)
    return out


@needs_lib
def test_no_kernel_breaks_a_rule(tmp_path):
    def check(co):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--mcpu=gfx950", co], check=True, capture_output=True,
                              text=True).stdout
        out = []
        for name, ins in functions(text, "").items():
            out += [(name, "barrier", hex(a)) for a in unwaited_barriers(ins)] if ins else []
            out += [(name, *pair) for pair in overwritten_stores(ins)]
        return out
    objs = code_objects(chasm.LIB_PATH, str(tmp_path))
    assert objs
    with cf.ThreadPoolExecutor(8) as ex:
        bad = [b for r in ex.map(check, objs) for b in r]
    assert not bad, (len(bad), bad[:20])


def test_the_store_rule_sees_the_next_instructions():
    store, over = "buffer_store_dwordx4 v[46:49], v114, s[16:19], s8 offen", "v_cvt_f64_u32_e32 v[48:49], v36"

    def code(*ops):
        return [(4 * i, op, None) for i, op in enumerate(ops)] + [(4 * len(ops), "s_endpgm", None)]
    assert overwritten_stores(code(store, over)) == [(store, over)]
    assert overwritten_stores(code(store, "s_nop 0", over)) == [(store, over)]
    assert overwritten_stores(code(store, "s_nop 1", over)) == []
    assert overwritten_stores(code(store, "v_add_f64 v[0:1], v[46:47], v[48:49]")) == []      # a read
    assert overwritten_stores(code("buffer_store_dwordx2 v[48:49], v0, s[16:19], 0 offen", over)) == []
    jump = [(0, store, None), (4, "s_branch 1", 12), (8, "s_endpgm", None), (12, over, None), (16, "s_endpgm", None)]
    assert overwritten_stores(jump) == [(store, over)]
