"""No kernel of the built library keeps registers in scratch memory: the metadata of
every gfx950 code object in libpx.so (AMDGPU note, private segment size per kernel)."""
import os
import struct

import pytest

from paper_2501_03061_amd import px

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    """The gfx950 ELF images of the offload bundles of a shared library."""
    at = lib.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", lib, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", lib, p)
            name = lib[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield lib[at + off:at + off + size]
        at = lib.find(MAGIC, at + len(MAGIC))


def _kernels(elf):
    """name -> scratch bytes per work item, from the NT_AMDGPU_METADATA note."""
    import msgpack
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for k in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + k * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + k * shentsize + 24)
        if kind != 7:  # SHT_NOTE
            continue
        p = off
        while p < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                for kern in msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]:
                    yield kern[".name"], kern[".private_segment_fixed_size"]
            p = desc + (descsz + 3) // 4 * 4


def test_no_kernel_uses_scratch():
    pytest.importorskip("msgpack")
    assert os.path.exists(px.LIB_PATH), "libpx.so is not built"
    with open(px.LIB_PATH, "rb") as f:
        lib = f.read()
    kernels = dict(k for elf in _code_objects(lib) for k in _kernels(elf))
    # every pass of the pair pipeline is there, on the largest cube with its energy among them
    for part in ("pass1_z", "pass2_xyIfLi96ELi96ELi96E", "pass3_z", "pass4_rows", "gemm_xhy_k", "gemm_xc_k"):
        assert any(part in k for k in kernels), part
    assert {k: v for k, v in kernels.items() if v} == {}


REMARKS = """a.hip:3:1: remark: Function Name: clean [-Rpass-analysis=kernel-resource-usage]
    3 | __global__ void clean() {
      | ^
a.hip:3:1: remark:     VGPRs: 128 [-Rpass-analysis=kernel-resource-usage]
a.hip:3:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:9:1: remark: Function Name: spills [-Rpass-analysis=kernel-resource-usage]
a.hip:9:1: remark:     ScratchSize [bytes/lane]: 12 [-Rpass-analysis=kernel-resource-usage]
"""


def test_build_refuses_scratch(monkeypatch, tmp_path):
    """The build fails, and links nothing, when the compiler reports scratch memory."""
    from paper_2501_03061_amd.csrc import build as b
    assert b.scratch_users(REMARKS) == {"spills": 12}

    class Done:
        returncode, stdout, stderr = 0, "", REMARKS

    calls = []
    monkeypatch.setattr(b.subprocess, "run", lambda cmd, **k: calls.append(cmd) or Done())
    monkeypatch.setattr(b, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(b, "OUT", str(tmp_path / "lib.so"))
    with pytest.raises(RuntimeError, match="scratch memory.*spills"):
        b.build(jobs=2)
    assert all("-shared" not in c for c in calls)
