"""What the built library's device code must not contain, whatever the compiler made of the sources: looked up in the
disassembly of libvitenc.so's own gfx950 code objects.  No GPU."""
import os
import re
import struct
import subprocess

import pytest

import paper_2502_00937_amd as V

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    """The gfx950 code objects in the library, one per source file."""
    path = os.path.join(os.path.dirname(V.__file__), "libvitenc.so")
    data = open(path, "rb").read()
    found, at = [], data.find(MAGIC)
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                found.append(data[at + offset:at + offset + size])
            p += 24 + length
        at = data.find(MAGIC, at + len(MAGIC))
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: its instructions, (address, text, address of a branch's target or None) each}"""
    out, d = {}, tmp_path_factory.mktemp("code")
    for i, blob in enumerate(_code_objects()):
        p = d / ("%d.co" % i)
        p.write_bytes(blob)
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", str(p)], check=True, text=True,
                              stdout=subprocess.PIPE).stdout
        name, start = None, 0
        for line in text.splitlines():
            if m := re.match(r"([0-9a-f]+) <(\S+)>:", line):
                start, name = int(m[1], 16), m[2]
                out[name] = []
            elif name and (m := re.match(r"\t(\S.*?)\s*// ([0-9A-F]+):[0-9A-F ]+(?:<\S+\+0x([0-9a-f]+)>)?", line)):
                out[name].append((int(m[2], 16), m[1], start + int(m[3], 16) if m[3] else None))
    return out


def _loads_to_lds(code):
    for i, (_, ins, _) in enumerate(code):
        if "_lds_" in ins.split()[0] and ins.startswith(("global_load", "buffer_load")):
            yield i, ins


def test_loads_to_lds_have_their_wait_states(kernels):
    """They are written as asm texts, so nobody but their author counts these for them: a load to LDS takes its destination from
    M0, one wait state behind a scalar write of it at the least, and its address from scalar registers, five behind a vector
    instruction that writes them."""
    loads = 0
    for name, code in kernels.items():
        for i, ins in _loads_to_lds(code):
            loads += 1
            assert not re.match(r"s_\w+ m0,", code[i - 1][1]), (name, code[i - 1], ins)
            base = re.search(r"s\[(\d+):(\d+)\]", ins)
            states, k = 0, i - 1
            while base and states < 5 and k >= 0:
                m = re.match(r"v_\w+ (?:s(\d+)|s\[(\d+):(\d+)\]),", code[k][1])
                if m:
                    lo, hi = (int(m[1]),) * 2 if m[1] else (int(m[2]), int(m[3]))
                    assert hi < int(base[1]) or lo > int(base[2]), (name, code[k], ins)
                nop = re.match(r"s_nop (\d+)", code[k][1])
                states, k = states + (int(nop[1]) + 1 if nop else 1), k - 1
    assert loads > 1000  # the matrix products' kernels were looked at


def _barriers_under_a_mask(code):
    """Barriers that a way through the code reaches between an instruction that narrows the execution mask to part of what it was
    (and keeps what it was in a register) and the one that gives it back."""
    index = {at: i for i, (at, _, _) in enumerate(code)}
    reg = r"(s\[\d+:\d+\]|vcc)"
    found, seen, todo = set(), set(), [(0, ())]
    while todo:
        i, masks = todo.pop()
        while i < len(code):
            at, ins, target = code[i]
            if m := re.match(r"s_(and|andn2|or)_saveexec_b64 %s, %s" % (reg, reg), ins):
                if m[1] == "or" and m[3] in masks:  # the other arm: the mask is given back, and narrowed behind this
                    masks = masks[:masks.index(m[3])]
                masks += (m[2],) if m[2] not in masks else ()
            elif (m := re.match(r"s_or_b64 exec, exec, %s" % reg, ins)) and m[1] in masks:
                masks = masks[:masks.index(m[1])]
            elif ins.startswith("s_barrier") and masks:
                found.add(at)
            if ins.startswith("s_endpgm"):
                break
            if target is not None:
                if (target, masks) not in seen:
                    seen.add((target, masks))
                    todo.append((index[target], masks))
                if ins.startswith("s_branch"):
                    break
            i += 1
    return found


def test_attention_barriers_are_under_no_mask(kernels):
    """A wave without query rows takes a path of its own, with as many barriers.  The choice has to be a scalar branch: chosen by
    the execution mask, both paths stand one behind the other in every wave's way, and whether a wave meets the other one's
    barriers, too, is the compiler's choice."""
    looked_at = 0
    for name, code in kernels.items():
        if "attention_bf16_kernel" not in name:
            continue
        looked_at += 1
        assert sum(ins.startswith("s_barrier") for _, ins, _ in code) >= 4, name
        assert not _barriers_under_a_mask(code), name
    assert looked_at >= 9


def test_no_kernel_keeps_registers_in_scratch_memory(kernels):
    assert not [(name, ins) for name, code in kernels.items() for _, ins, _ in code if ins.startswith("scratch_")]
