"""Registers of the built kernels, from the metadata of the library's own code
objects: the kernels that run over pairs keep everything in registers (a spill in
their loops is memory traffic per pair)."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2208_14639_amd", "libvv10.so")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(tmp):
    """{kernel name: {metadata field: value}} over the library's gfx950 code objects."""
    fat = os.path.join(tmp, "fatbin")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", f".hip_fatbin={fat}", LIB,
                    os.path.join(tmp, "copy")], check=True)
    data, out, at = open(fat, "rb").read(), {}, 0
    while (at := data.find(MAGIC, at)) >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, pos - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" not in name or size == 0:
                continue
            obj = os.path.join(tmp, "object")
            with open(obj, "wb") as f:
                f.write(data[at + off:at + off + size])
            notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], check=True,
                                   capture_output=True, text=True).stdout
            for part in notes.split("  - .agpr_count:")[1:]:
                fields = dict(re.findall(r"\.([a-z_]+):\s+(\S+)", part))
                out[fields["symbol"]] = fields
        at = pos
    return out


needs_llvm = pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-readelf")),
                                reason="no llvm tools")


@needs_llvm
@pytest.mark.parametrize("name,count", [("k_grid", 10), ("k_w?contract", 60), ("k_pair", 4)])
def test_pair_kernels_do_not_spill(tmp_path, name, count):
    found = {k: v for k, v in kernels(str(tmp_path)).items() if re.search(name, k)}
    assert len(found) >= count
    spilled = {k: v["vgpr_spill_count"] for k, v in found.items() if int(v["vgpr_spill_count"])}
    assert not spilled, spilled
