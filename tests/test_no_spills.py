"""No kernel of the built librfq.so keeps values in scratch memory: a launch
bound that leaves a kernel too few registers costs more than the waves it
gains (64 rows x 4096 x 2880: 7.5 us with 15 registers spilled, 6.7 without)."""
import re
import struct
import subprocess

from paper_2608_26581_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(data):
    """The gfx950 code objects in the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if size and target.endswith(b"gfx950"):
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 1)


def _kernels(path, tmp_path):
    with open(path, "rb") as f:
        data = f.read()
    for i, obj in enumerate(_code_objects(data)):
        file = tmp_path / ("%d.elf" % i)
        file.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(file)], capture_output=True, text=True,
                               check=True).stdout
        for k in re.split(r"\n\s+- \.a(?:gpr_count|rgs):", notes)[1:]:
            name = re.search(r"\.name:\s+(_Z\w+)", k).group(1)
            yield name, {f: int(re.search(r"\.%s:\s+(\d+)" % f, k).group(1))
                         for f in ("private_segment_fixed_size", "vgpr_spill_count")}


def test_no_kernel_uses_scratch(tmp_path):
    kernels = dict(_kernels(build.LIB_PATH, tmp_path))
    assert any("rfq_gemm_skinny_kernel" in k for k in kernels)
    assert any("hif4_gemm_kernel" in k for k in kernels)
    assert {k: v for k, v in kernels.items() if any(v.values())} == {}
