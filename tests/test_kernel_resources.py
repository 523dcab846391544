"""How many workgroups of a kernel share a CU, from the register counts and LDS that its code object states (built library, no GPU)."""
import os
import re
import struct
import subprocess

import pytest
import yaml

from paper_2602_21233_amd import build

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """mangled name -> metadata of every kernel in the library's gfx950 code objects"""
    lib = open(build.LIB if os.path.exists(build.LIB) else build.build_library(), "rb").read()
    folder, found = tmp_path_factory.mktemp("code"), {}
    at = lib.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", lib, at + len(MAGIC))[0]):
            start, size, n = struct.unpack_from("<QQQ", lib, pos)
            if b"gfx950" in lib[pos + 24:pos + 24 + n]:
                (folder / "code").write_bytes(lib[at + start:at + start + size])
                notes = subprocess.run([READELF, "--notes", str(folder / "code")], check=True, capture_output=True, text=True).stdout
                text = notes[notes.index("---"):notes.rindex("\n...")]
                for k in yaml.load(text, Loader=getattr(yaml, "CSafeLoader", yaml.SafeLoader))["amdhsa.kernels"]:
                    found[k[".name"]] = k
            pos += 24 + n
        at = lib.find(MAGIC, at + 1)
    return found


# A batch of short prompts is up to 2048 workgroups of the small call's kernel: as many of them share a CU as its 160 KB of LDS hold.
# Registers: 512 a lane of a SIMD, in steps of 8; a workgroup is two wavefronts on each of the four SIMDs.
@pytest.mark.parametrize("D,lds_kb", [(64, 53), (128, 67)])
@pytest.mark.parametrize("Bs", [64, 128])
@pytest.mark.parametrize("ext", [0, 1])
def test_workgroups_of_small_calls_share_a_cu(kernels, D, lds_kb, Bs, ext):
    name, = [n for n in kernels if re.search(rf"score_topk_small_kernelILi{D}ELi{Bs}ELb{ext}E", n)]
    k = kernels[name]
    assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0
    wavefronts = 512 // (-(-k[".vgpr_count"] // 8) * 8)
    assert wavefronts // 2 >= 160 // lds_kb, k[".vgpr_count"]
