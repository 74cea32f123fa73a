"""Every barrier of the cube kernels comes after a wait for the wave's own LDS accesses
(lgkmcnt(0)) on every path that reaches it: without one, another wave can pass the barrier
and read LDS that has not been written yet.  The paths include loops' back edges, where the
compiler has left the wait out.  Checked on the gfx950 code of the compiled units, where
they are present."""
import concurrent.futures as cf
import glob
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"
OBJECTS = sorted(p for n in (8, 16, 24, 32) for p in glob.glob(os.path.join(ROOT, "_build", "obj", f"inst_*_n{n}_*_c0.hip.o")))


def functions(text, kernel):
    """name -> [(address, instruction, branch target or None)] of the functions named after
    kernel, addresses from the function's start."""
    out, cur, base = {}, None, 0
    blocks = [b for b in text.split("\n\n") if kernel in b.split("\n", 1)[0]]
    for line in "\n".join(blocks).splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if m:
            base, cur = int(m.group(1), 16), out.setdefault(m.group(2), [])
            continue
        m = re.match(r"^\s+(.+?)\s*//\s*([0-9A-F]+):(.*)$", line)
        if m and cur is not None:
            t = re.search(r"<[^+>]+(?:\+0x([0-9a-f]+))?>", m.group(3))
            cur.append((int(m.group(2), 16) - base, m.group(1).strip(), (int(t.group(1) or "0", 16) if t else None)))
    return out


def unwaited_barriers(ins):
    """Addresses of barriers that some path reaches with LDS accesses outstanding."""
    at = {a: i for i, (a, _, _) in enumerate(ins)}
    pending, seen, work, bad = [False] * len(ins), [False] * len(ins), [0], set()
    seen[0] = True
    while work:
        i = work.pop()
        a, op, target = ins[i]
        p = pending[i]
        if op.startswith("s_barrier") and p:
            bad.add(a)
        if op.startswith("ds_") and not op.startswith(("ds_bpermute", "ds_permute", "ds_swizzle")):
            p = True
        if op.startswith("s_waitcnt") and "lgkmcnt(0)" in op:
            p = False
        nxt = []
        if op.startswith(("s_branch", "s_cbranch")) and target in at:
            nxt.append(at[target])
        if not op.startswith(("s_branch", "s_endpgm")) and i + 1 < len(ins):
            nxt.append(i + 1)
        for j in nxt:
            if not seen[j] or (p and not pending[j]):
                seen[j] = True
                pending[j] = pending[j] or p
                work.append(j)
    return sorted(bad)


def device_code(obj, tmp):
    fat, co = os.path.join(tmp, os.path.basename(obj) + ".fb"), os.path.join(tmp, os.path.basename(obj) + ".co")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", obj, fat + ".o"], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={co}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    return subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--mcpu=gfx950", co], check=True, capture_output=True, text=True).stdout


def test_the_check_sees_a_back_edge_without_a_wait():
    loop = [(0, "s_waitcnt lgkmcnt(0)", None), (4, "s_barrier", None), (8, "ds_read_b32 v0, v1", None),
            (16, "s_waitcnt lgkmcnt(0)", None), (20, "ds_write_b32 v1, v0", None), (28, "s_cbranch_scc1 65529", 4),
            (32, "s_endpgm", None)]
    assert unwaited_barriers(loop) == [4]
    loop[5] = (28, "s_cbranch_scc1 65528", 0)            # through the wait
    assert unwaited_barriers(loop) == []


@pytest.mark.skipif(not OBJECTS or not os.path.exists(f"{LLVM}/clang-offload-bundler"), reason="no compiled units")
def test_no_barrier_with_outstanding_lds_accesses(tmp_path):
    def check(obj):
        return [(os.path.basename(obj), name, a) for name, ins in functions(device_code(obj, str(tmp_path)), "k_cube").items() if ins
                for a in unwaited_barriers(ins)]
    with cf.ThreadPoolExecutor(8) as ex:
        bad = [b for r in ex.map(check, OBJECTS) for b in r]
    assert not bad, bad
