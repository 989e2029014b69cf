"""Registers and scratch memory of the kernels in the built library, as the compiler left them in its metadata."""
import os
import re
import struct
import subprocess

import pytest

from paper_2503_08640_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(tmp_path):
    """[(mangled name, {field: value})] of every gfx950 kernel in the library."""
    with open(build.LIB_PATH, "rb") as f:
        data = f.read()
    found = []
    for n, at in enumerate(m.start() for m in re.finditer(b"\x7fELF\x02\x01\x01", data)):
        if struct.unpack_from("<H", data, at + 18)[0] != 224:  # e_machine: AMDGPU
            continue
        path = tmp_path / f"object{n}"
        # (a code object ends somewhere behind its section headers; what follows it in the library does not matter)
        path.write_bytes(data[at:])
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for part in re.split(r"^  - (?=\.a)", notes, flags=re.M)[1:]:
            fields = dict(re.findall(r"^    (\.\w+): +(\S+)$", part, flags=re.M))
            if ".name" in fields:
                found.append((fields[".name"], fields))
    return found


@pytest.mark.skipif(not (os.path.exists(READELF) and os.path.exists(build.LIB_PATH)), reason="needs the built library and llvm-readelf")
def test_no_pipelined_kernel_keeps_registers_in_scratch(tmp_path):
    """A reload from scratch inside a tile loop waits for every tile load in flight."""
    found = [x for x in kernels(tmp_path) if "attn_prefill" in x[0] or "decode_group" in x[0]]
    assert sum("attn_prefill64_kernel" in name for name, _ in found) >= 30 and any("decode_group_kernel" in name for name, _ in found)
    spilled = {name: (f[".vgpr_spill_count"], f[".private_segment_fixed_size"]) for name, f in found
               if f[".vgpr_spill_count"] != "0" or f[".private_segment_fixed_size"] != "0"}
    assert not spilled
