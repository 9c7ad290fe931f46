"""Registers of the built kernels, from the code objects' own metadata: no
kernel spills a vector register or uses scratch memory, and the grouped-head
builds keep the waves per SIMD that the launch rules count with."""

import os
import re
import struct
import subprocess

import pytest

from paper_2609_19702_amd import binding as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The GPU code objects of every offload bundle in a library's bytes."""
    at = data.find(MAGIC)
    while at >= 0:
        (count,), p = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            name, p = data[p + 24:p + 24 + n], p + 24 + n
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    B.lib()
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    found = {}
    for i, co in enumerate(code_objects(data)):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True,
                               text=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            name = re.search(r"\.symbol:\s+(\S+)\.kd", k).group(1)
            found[name] = {f: int(re.search(rf"\.{f}:\s+(\d+)", k).group(1))
                           for f in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    return found


def test_no_kernel_spills(kernels):
    assert len(kernels) > 90
    bad = {n: k for n, k in kernels.items() if k["vgpr_spill_count"] or k["private_segment_fixed_size"]}
    assert not bad


def test_plan_driven_fp8_grouped_heads_keep_four_waves_per_simd(kernels):
    # decode_mfma_kernel<KvFp8, D, G, FUSED = false, Kept, ONE>: d = 64, and the
    # build of one tile in flight
    seen = {n: k["vgpr_count"] for n, k in kernels.items()
            if re.search(r"decode_mfma_kernel.*KvFp8E(Li64E.*Lb0E.*Lb0E|Li128E.*Lb0E.*Lb1E)", n)}
    assert len(seen) == 6 and max(seen.values()) <= 128, seen


def test_grouped_head_waves_per_cu(kernels):
    """The launch rule's waves per CU (four SIMDs of 512 registers): 8 of d = 128
    and 12 of d = 64."""
    for d, waves in ((128, 8), (64, 12)):
        seen = [k["vgpr_count"] for n, k in kernels.items()
                if "decode_mfma_kernel" in n and f"Li{d}E" in n]
        assert len(seen) == (27 if d == 128 else 24) and max(seen) <= 512 // (waves // 4) // 8 * 8
