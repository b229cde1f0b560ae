"""Registers and scratch memory of built kernels, from the library's own code objects."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2605_28451_amd import _lib

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(tmp_path):
    """{mangled name: (VGPRs, scratch bytes per lane)} of every gfx950 kernel."""
    if not (os.path.exists(_lib.LIB_PATH) and os.path.exists(READELF)):
        pytest.skip("needs the built library and llvm-readelf")
    data, found, at = open(_lib.LIB_PATH, "rb").read(), {}, -1
    while (at := data.find(BUNDLE, at + 1)) >= 0:
        count, pos = struct.unpack_from("<Q", data, at + len(BUNDLE))[0], at + len(BUNDLE) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" in target and size:
                (tmp_path / "code").write_bytes(data[at + offset:at + offset + size])
                notes = subprocess.run([READELF, "--notes", str(tmp_path / "code")], capture_output=True,
                                       text=True, check=True).stdout
                for entry in notes.split("  - .agpr_count:")[1:]:
                    field = {k: re.search(rf"\.{k}:\s+(\S+)", entry).group(1)
                             for k in ("name", "vgpr_count", "private_segment_fixed_size")}
                    found[field["name"]] = (int(field["vgpr_count"]), int(field["private_segment_fixed_size"]))
    return found


def test_large_half_precision_forward_transforms_fit_two_workgroups(tmp_path):
    # 1024 threads of at most 64 registers: two workgroups per CU, without
    # scratch (row_kernel and row_kernel_rr<..., 1 row, ..., plan 1>, LOG2N = 14,
    # OP_FWD, with storage and FP32 outputs)
    names = kernels(tmp_path)
    pick = {k: v for k, v in names.items()
            if re.search(r"row_kernel(_rr)?INS_\d+Mode(FP16|F16Mul\w*)ELi14ELi0ELi0E", k)}
    assert len(pick) >= 6, sorted(pick)
    assert all(vgprs <= 64 and scratch == 0 for vgprs, scratch in pick.values()), pick


def test_large_pure_half_precision_inverses_fit_two_workgroups(tmp_path):
    # the same for the pure-FP16 inverse and for the output-phase adjoint
    names = kernels(tmp_path)
    pick = {k: v for k, v in names.items()
            if re.search(r"row_kernel(_rr)?INS_8ModeFP16ELi14ELi(1ELi[02]E|2ELi13[24]E)", k)
            and not re.search(r"row_kernel_rrINS_8ModeFP16ELi14ELi1ELi[02]ELb0ELi2E", k)}
    assert len(pick) >= 6, sorted(pick)
    assert all(vgprs <= 64 and scratch == 0 for vgprs, scratch in pick.values()), pick
