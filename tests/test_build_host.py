"""Host-side checks of the build script's incremental rule and of what the built kernels hold (no compiler is run)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2212_05191_amd import build as B


def _touch(path, mtime):
    with open(path, "w") as f:
        f.write("x")
    os.utime(path, (mtime, mtime))


def test_incremental_build_recompiles_objects_older_than_a_header(tmp_path):
    # objects share struct layouts through the headers: one compiled before a header changed must not be linked
    srcs = ["a.hip", "b.hip", "c.hip", "d.hip"]
    objs = [str(tmp_path / s.replace(".hip", ".o")) for s in srcs]
    old_h, new_h = str(tmp_path / "old.hpp"), str(tmp_path / "new.hpp")
    _touch(old_h, 1000)
    _touch(new_h, 2000)
    _touch(objs[0], 1500)    # asked for anyway
    _touch(objs[1], 1500)    # older than new.hpp: stale
    _touch(objs[2], 2500)    # newer than every header: kept
    # objs[3] does not exist: compiled
    got = B.sources_to_compile(["a.hip"], srcs, objs, [old_h, new_h])
    assert got[0] == "a.hip" and sorted(got) == ["a.hip", "b.hip", "d.hip"]


def test_incremental_build_keeps_fresh_objects_and_passes_other_names_through(tmp_path):
    srcs = ["a.hip", "b.hip"]
    objs = [str(tmp_path / "a.o"), str(tmp_path / "b.o")]
    hdr = str(tmp_path / "h.hpp")
    _touch(hdr, 1000)
    _touch(objs[0], 2000)
    _touch(objs[1], 2000)
    assert B.sources_to_compile(["peaks_probe.hip"], srcs, objs, [hdr]) == ["peaks_probe.hip"]
    assert B.sources_to_compile([], srcs, objs, [hdr]) == []
    os.utime(hdr, (3000, 3000))
    assert sorted(B.sources_to_compile([], srcs, objs, [hdr])) == ["a.hip", "b.hip"]


def test_every_source_of_the_library_exists_and_every_hip_file_is_built():
    on_disk = {f for f in os.listdir(B.CSRC) if f.endswith(".hip")}
    assert set(B.SOURCES) | {"peaks_probe.hip"} == on_disk
    assert "-packed-fp32-ops" in B.FLAGS and "--offload-arch=gfx950" in B.FLAGS


def _kernel_resources(tmp_path):
    """Kernel symbol -> (LDS bytes, vector registers), from the metadata notes of the device code in the built library."""
    readelf = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
    if not (os.path.exists(B.LIB) and os.path.exists(readelf)):
        pytest.skip("needs the built library and llvm-readelf")
    blob, magic, found, at = open(B.LIB, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}, 0
    while (at := blob.find(magic, at)) >= 0:     # magic, entries, then of each: offset, size, length of the target's name, name
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, pos - 8)[0]):
            offset, size, length = struct.unpack_from("<3Q", blob, pos)
            target, pos = blob[pos + 24:pos + 24 + length], pos + 24 + length
            if b"gfx950" in target:
                (tmp_path / "code").write_bytes(blob[at + offset:at + offset + size])
                notes = subprocess.run([readelf, "--notes", str(tmp_path / "code")], stdout=subprocess.PIPE, text=True, check=True).stdout
                for k in notes.split(".agpr_count:")[1:]:
                    field = {f: re.search(rf"\.{f}:\s+(\S+)", k)[1] for f in ("name", "group_segment_fixed_size", "vgpr_count")}
                    found[field["name"]] = int(field["group_segment_fixed_size"]), int(field["vgpr_count"])
        at += len(magic)
    return found


def test_a_router_gradient_kernel_of_one_part_holds_that_part_only(tmp_path):
    """The kernel of the token gradient for two chunks of logit columns leaves room for four workgroups of four waves on a CU (160 KB of LDS, 512
    registers a SIMD lane); with the LDS of the router weights it had 46 KB and 136 registers, three."""
    res = _kernel_resources(tmp_path)
    (lds, regs), = [v for k, v in res.items() if "router_grad_mfma_kernelILi2ELi0E" in k]
    assert lds == 256 * (2 * 16 + 8) * 2 + 4 * 32 * 9 * 16 and 4 * lds <= 160 * 1024    # transposed weights, rows of x
    assert regs <= 512 // 4
