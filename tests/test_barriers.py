"""No barrier of a kernel may be reached while the wave's own shared-memory
accesses are in flight: the waves that the barrier lets go on would read old
values, or write over what is still being read.  The compiler inserts the wait,
and loses it at some loop heads, so the built code itself is looked over: a
forward data flow over each kernel's control flow graph, from the disassembly of
the gfx950 code in libtla.so."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2609_36529_amd as tla

OBJDUMP = next((p for p in (shutil.which("llvm-objdump"), "/opt/rocm/lib/llvm/bin/llvm-objdump",
                            "/opt/rocm/llvm/bin/llvm-objdump") if p and os.path.exists(p)), None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects of the offload bundles inside a shared library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n if n < 16 else 0):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def kernels(text):
    """(name, [(address, instruction, branch target or None)]) of a disassembly."""
    name, base, ins = None, 0, []
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            if ins:
                yield name, ins
            name, base, ins = m.group(2), int(m.group(1), 16), []
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):(.*)$", line)
        if m:
            t = re.search(r"<[^>+]+(?:\+0x([0-9a-f]+))?>", m.group(3))
            target = base + int(t.group(1) or "0", 16) if t else None
            ins.append((int(m.group(2), 16), m.group(1), target))
    if ins:
        yield name, ins


def in_flight_at_barriers(ins):
    """Addresses of the barriers that some path reaches with shared-memory
    accesses issued since the last wait for all of them."""
    index = {a: i for i, (a, _, _) in enumerate(ins)}
    state, bad, work = {0: False}, set(), [0]
    while work:
        i = work.pop()
        pending = state[i]
        addr, s, target = ins[i]
        op = s.split()[0]
        if op == "s_barrier" and pending:
            bad.add(addr)
        elif op.startswith("ds_") and not re.search(r"permute|swizzle", op):
            pending = True
        elif op == "s_waitcnt" and ("lgkmcnt(0)" in s or "cnt" not in s.split(None, 1)[1]):
            pending = False
        nxt = [] if op in ("s_endpgm", "s_branch") else [i + 1]
        if op == "s_branch" or op.startswith("s_cbranch"):
            nxt.append(index[target])
        for j in nxt:
            if j < len(ins) and (j not in state or (pending and not state[j])):
                state[j] = state.get(j, False) or pending
                work.append(j)
    return bad


def test_the_data_flow():
    """Listings by hand: an access waited for, one that only the loop's way back
    leaves in flight, and one on a path of its own."""
    b, e = "s_barrier", "s_endpgm"
    wait = "s_waitcnt lgkmcnt(0)"

    def seq(*ops):
        return [(4 * i, *(o if isinstance(o, tuple) else (o, None))) for i, o in enumerate(ops)]

    st = "ds_write_b32 v0, v1"
    assert in_flight_at_barriers(seq(st, wait, b, e)) == set()
    assert in_flight_at_barriers(seq(st, "s_waitcnt lgkmcnt(1)", b, e)) == {8}
    assert in_flight_at_barriers(seq(b, st, ("s_cbranch_scc1 65533", 0), wait, b, e)) == {0}
    assert in_flight_at_barriers(seq(("s_cbranch_scc0 1", 8), st, b, e)) == {8}
    assert in_flight_at_barriers(seq("ds_read_b32 v0, v1", b, e)) == {4}
    assert in_flight_at_barriers(seq("ds_bpermute_b32 v0, v1, v2", b, e)) == set()


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_nothing_in_flight_at_a_barrier(tmp_path):
    seen = 0
    for n, obj in enumerate(code_objects(tla.LIB_PATH)):
        f = tmp_path / f"{n}.co"
        f.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", str(f)], capture_output=True, text=True, check=True).stdout
        for name, ins in kernels(text):
            seen += any(s.startswith("s_barrier") for _, s, _ in ins)
            bad = in_flight_at_barriers(ins)
            assert not bad, (name, [hex(a) for a in sorted(bad)])
    assert seen > 100, seen
