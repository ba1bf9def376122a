"""The code the compiler made of the kernels (CPU-only: the built library's
device code, disassembled): properties that the sources rely on and that no
result shows reliably."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_1912_11554_amd as nuts

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_objects(path):
    """The gfx950 code objects bundled in a host library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        count = struct.unpack_from("<Q", data, at + len(MAGIC))[0]
        entry = at + len(MAGIC) + 8
        for _ in range(count if count < 16 else 0):  # (else the magic stands in host code)
            off, size, idlen = struct.unpack_from("<QQQ", data, entry)
            ident = data[entry + 24:entry + 24 + idlen]
            entry += 24 + idlen
            if b"gfx950" in ident:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _functions(obj, tmp):
    """{symbol: [instruction text]} of one code object."""
    path = os.path.join(tmp, "object")
    with open(path, "wb") as f:
        f.write(obj)
    out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], check=True, capture_output=True,
                         text=True).stdout
    funcs, cur = {}, None
    for line in out.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        if m:
            cur = funcs.setdefault(m.group(1), [])
        elif cur is not None and line.startswith("\t"):
            cur.append(line.split("//")[0].strip())
    return funcs


needs_objdump = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")


@needs_objdump
def test_buffer_resources_are_uniform(tmp_path):
    # a buffer access from a resource that differs between the lanes becomes a
    # loop over the distinct resources (the lanes narrowed, the access, the
    # lanes done taken out, back to the start)
    seen, loops = 0, []
    for obj in _device_objects(nuts.LIB_PATH):
        if b"sampler_batch_kernel" not in obj:
            continue
        for name, ins in _functions(obj, str(tmp_path)).items():
            if "sampler_batch_kernel" not in name:
                continue
            seen += 1
            for i, text in enumerate(ins):
                if re.match(r"buffer_(load|store)", text):
                    after = ins[i + 1:i + 6]
                    if any(t.startswith("s_xor_b64 exec, exec") for t in after) and \
                            any(t.startswith("s_cbranch_execnz") for t in after):
                        loops.append((name, text))
    assert seen == 22  # every instantiation: 11 shapes, with and without the optional features
    assert not loops, loops[:4]


@needs_objdump
def test_evaluators_stay_in_registers(tmp_path):
    # a function that takes an evaluator by reference and is not inlined keeps
    # it in scratch memory for the whole chain
    kernels, others = 0, []
    for obj in _device_objects(nuts.LIB_PATH):
        if b"sampler_hmm_kernel" not in obj and b"sampler_wave_kernel" not in obj and \
                b"sampler_grid_kernel" not in obj and b"sampler_team_kernel" not in obj and \
                b"sampler_batch_kernel" not in obj:
            continue
        for name in _functions(obj, str(tmp_path)):
            kernels += "_kernel" in name
            if re.search(r"(Hmm|Wave|Grid|Batch)Eval", name):
                others.append(name)
    assert kernels > 100
    assert not others, others
