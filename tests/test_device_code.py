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
    """{mangled kernel name: its instructions, one text each}"""
    out, d = {}, tmp_path_factory.mktemp("code")
    for i, blob in enumerate(_code_objects()):
        p = d / ("%d.co" % i)
        p.write_bytes(blob)
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", str(p)], check=True, text=True,
                              stdout=subprocess.PIPE).stdout
        name = None
        for line in text.splitlines():
            if m := re.match(r"[0-9a-f]+ <(\S+)>:", line):
                name = m[1]
                out[name] = []
            elif name and line.startswith("\t"):
                out[name].append(line.split("//")[0].strip())
    return out


def _loads_to_lds(code):
    for i, ins in enumerate(code):
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
            assert not re.match(r"s_\w+ m0,", code[i - 1]), (name, code[i - 1], ins)
            base = re.search(r"s\[(\d+):(\d+)\]", ins)
            states, k = 0, i - 1
            while base and states < 5 and k >= 0:
                m = re.match(r"v_\w+ (?:s(\d+)|s\[(\d+):(\d+)\]),", code[k])
                if m:
                    lo, hi = (int(m[1]),) * 2 if m[1] else (int(m[2]), int(m[3]))
                    assert hi < int(base[1]) or lo > int(base[2]), (name, code[k], ins)
                nop = re.match(r"s_nop (\d+)", code[k])
                states, k = states + (int(nop[1]) + 1 if nop else 1), k - 1
    assert loads > 1000  # the matrix products' kernels were looked at
