"""What the built kernels take of a compute unit, read from the library's own metadata (no GPU needed).  Up to 128 vector
registers leave room for two workgroups of 8 wavefronts on one compute unit; one more halves what is in flight."""
import os
import re
import struct
import subprocess

import pytest

import paper_2412_07174_amd as scap

READOBJ = "/opt/rocm/llvm/bin/llvm-readobj"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: {field: value}} of every gfx950 kernel in the library."""
    if not os.path.exists(READOBJ):
        pytest.skip("no llvm-readobj")
    if not os.path.exists(scap.lib_path()):
        from paper_2412_07174_amd import build
        build.build(verbose=False)
    lib = open(scap.lib_path(), "rb").read()
    path = str(tmp_path_factory.mktemp("code") / "object")
    found, at = {}, lib.find(MAGIC)
    while at >= 0:
        (entries,) = struct.unpack_from("<Q", lib, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", lib, pos)
            target = lib[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" not in target or size == 0:
                continue
            with open(path, "wb") as f:
                f.write(lib[at + offset:at + offset + size])
            notes = subprocess.run([READOBJ, "--notes", path], check=True, stdout=subprocess.PIPE, text=True).stdout
            for text in notes.split(".agpr_count")[1:]:
                name = re.search(r"\.name:\s+(_Z\w+)", text)
                if name:
                    found[name.group(1)] = {k: int(re.search(rf"\.{k}:\s+(\d+)", text).group(1))
                                            for k in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
        at = lib.find(MAGIC, at + 1)
    names = subprocess.run(["c++filt"], input="\n".join(found), check=True, stdout=subprocess.PIPE, text=True).stdout.split("\n")
    return {re.sub(r"^void |\(.*", "", n): v for n, v in zip(names, found.values())}


def _of(kernels, pattern):
    some = {n: v for n, v in kernels.items() if re.fullmatch(pattern, n)}
    assert some, pattern
    return some


def test_value_lists_of_3_to_4_tokens_leave_room_for_two_workgroups(kernels):
    """int8 and bf16 weights, input prologue (plain and gating): their launches are planned for two per compute unit."""
    for name, r in _of(kernels, r"scap::gemm_inline_kernel<[12], 4, [01]>").items():
        assert r["vgpr_count"] <= 128, (name, r)


def test_staged_tile_leaves_room_for_two_workgroups(kernels):
    """16-bit weights and 8-byte int8 lanes."""
    for name, r in _of(kernels, r"scap::gemm_inline_raw_kernel<[013], [01], false, (true|false), \d>").items():
        assert r["vgpr_count"] <= 128, (name, r)


def test_row_steps_leave_room_for_two_workgroups_where_the_plan_counts_on_it(kernels):
    """Inputs that are the operand, whole octets, 16-bit weights; all forms of 8-byte int8 lanes."""
    for name, r in _of(kernels, r"scap::gemm_rows_kernel<([01], [01], 0, false|3, [01], \d, (true|false)), \d+>").items():
        assert r["vgpr_count"] <= 128, (name, r)


def test_batch_kernels_keep_everything_in_registers(kernels):
    for name, r in _of(kernels, r"scap::gemm_(inline|inline_raw|rows)_kernel<.*>").items():
        assert r["private_segment_fixed_size"] == 0 and r["vgpr_spill_count"] == 0, (name, r)
