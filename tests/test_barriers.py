"""CPU-only check of the built library's gfx950 code: at every workgroup barrier, on every path that leads to it, the wave
has waited for its own LDS accesses.  What one wave stores before a barrier is otherwise not certain to be there
for the waves that read it after the barrier; two instructions of difference in the code decide whether that is ever seen."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def code_objects(path):
    """The device ELF images inside a library that hipcc linked."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name]:
                yield data[at + offset:at + offset + size]
            p += 24 + name
        at = data.find(magic, at + 1)


def kernels(text):
    """{name: [(address, instruction, branch target or None)]} of a disassembly."""
    out, name = {}, None
    for line in text.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:$", line)
        if m:
            name = out.setdefault(m.group(1), [])
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+): ", line)
        if m and name is not None:
            at, ins, to = int(m.group(2), 16), m.group(1), None
            b = re.match(r"s_c?branch\S*\s+(\d+)", ins)
            if b:
                words = int(b.group(1))
                to = at + 4 + 4 * (words - 65536 if words >= 32768 else words)
            name.append((at, ins, to))
    return out


def outstanding_at_barriers(code):
    """(barriers, those of them at which an LDS access can be outstanding).  Every path is followed."""
    index = {at: i for i, (at, _, _) in enumerate(code)}
    seen, bad, work = [0] * len(code), set(), [(0, 1)]        # bits: reached with nothing outstanding, with something
    while work:
        i, state = work.pop()
        while i < len(code) and not seen[i] & state:
            seen[i] |= state
            _, ins, to = code[i]
            op = ins.split()[0]
            if op.startswith("ds_") and not op.startswith(("ds_bpermute", "ds_permute", "ds_swizzle", "ds_nop")):
                state = 2
            elif op == "s_waitcnt" and ("lgkmcnt(0)" in ins or ins.split()[1:] == ["0"]):
                state = 1
            elif op == "s_barrier" and state == 2:
                bad.add(i)
            if to is not None:
                work.append((index[to], state))
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            i += 1
    return sum(ins.startswith("s_barrier") for _, ins, _ in code), sorted(bad)


def test_the_check_follows_loops():
    store, wait, barrier = (0, "ds_write_b32 v0, v1", None), (0, "s_waitcnt lgkmcnt(0)", None), (0, "s_barrier", None)

    def program(*parts):
        return [(4 * i, ins, to) for i, (_, ins, to) in enumerate(parts)]
    back = (0, "s_cbranch_scc1 0", 0)
    end = (0, "s_endpgm", None)
    assert outstanding_at_barriers(program(wait, barrier, store, end)) == (1, [])
    assert outstanding_at_barriers(program(store, wait, barrier, end)) == (1, [])
    assert outstanding_at_barriers(program(store, barrier, end)) == (1, [1])
    assert outstanding_at_barriers(program(barrier, store, back, end)) == (1, [0])        # round the loop
    assert outstanding_at_barriers(program(wait, barrier, store, back, end)) == (1, [])
    assert outstanding_at_barriers(program((0, "s_cbranch_scc0 1", 8), wait, barrier, end)) == (1, [])
    assert outstanding_at_barriers(program(store, (0, "s_cbranch_scc0 1", 12), wait, barrier, end)) == (1, [3])


def test_waves_wait_for_their_lds_accesses_before_every_barrier():
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler in this installation")
    from paper_2508_17828_amd import trim
    if not os.path.exists(trim.LIB_PATH):
        from paper_2508_17828_amd import build
        build.build()
    barriers, bad = 0, {}
    with tempfile.TemporaryDirectory() as tmp:
        for i, image in enumerate(code_objects(trim.LIB_PATH)):
            p = os.path.join(tmp, f"{i}.o")
            with open(p, "wb") as f:
                f.write(image)
            text = subprocess.run([OBJDUMP, "-d", p], check=True, capture_output=True, text=True).stdout
            for name, code in kernels(text).items():
                n, at = outstanding_at_barriers(code)
                barriers += n
                if at:
                    bad[name] = len(at)
    assert barriers > 1000
    assert not bad, f"{len(bad)} kernels, {sum(bad.values())} barriers: {sorted(bad.items())[:4]}"
