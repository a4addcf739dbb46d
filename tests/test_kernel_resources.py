"""The built kernels' registers, LDS and scratch, read from the library's own
code object: how many waves of a launch share a CU (512 vector registers per
lane of a SIMD in steps of 8, 160 KB of LDS, 8 waves per SIMD)."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2103_10765_amd import gbm3d

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 ELF images of the library's offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                yield data[at + off:at + off + size]
            p += 24 + length
        at = data.find(MAGIC, at + 1)


def _metadata(elf):
    """The kernels of the AMDGPU metadata note (owner AMDGPU, type 32)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        h = struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * size)
        if h[1] != 7:
            continue
        p, end = h[4], h[4] + h[5]
        while p < end:
            ns, ds, kind = struct.unpack_from("<III", elf, p)
            body = p + 12 + (ns + 3) // 4 * 4
            if kind == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[body:body + ds], strict_map_key=False)["amdhsa.kernels"]
            p = body + (ds + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(gbm3d.LIB_PATH):
        pytest.fail("libgbm3d.so is not built (run __graft_entry__.build())")
    found = [k for e in _code_objects(open(gbm3d.LIB_PATH, "rb").read()) for k in _metadata(e)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    out = {}
    for name, k in zip(names, found):
        name = re.sub(r"\(gbm3d::\w+\)", "", name.replace("(anonymous namespace)::", ""))
        out[re.search(r"(\w+(<[^(]*>)?)\(", name).group(1)] = k
    return out


def waves_per_cu(k):
    waves = k[".max_flat_workgroup_size"] // 64
    per_simd = min(8, 512 // (-(-k[".vgpr_count"] // 8) * 8))
    return min(160 * 1024 // max(k[".group_segment_fixed_size"], 1), 4 * per_simd // waves) * waves


@pytest.mark.parametrize("variant", ["false, false", "false, true", "true, false"])
def test_first_stage_groups_of_32_share_a_cu(kernels, variant):
    """The hard-threshold kernel at K = 32, single image, from pixels and batch:
    24 waves per CU, nothing in scratch memory."""
    k = kernels[f"group_ht_kernel<32, {variant}, 0>"]
    assert waves_per_cu(k) >= 24 and k[".private_segment_fixed_size"] == 0


@pytest.mark.parametrize("K", [2, 4, 8, 16])
@pytest.mark.parametrize("batch", ["false", "true"])
def test_second_stage_groups_of_up_to_16_fill_a_cu(kernels, K, batch):
    """The Wiener kernel at K <= 16, single image and batch: 32 waves per CU
    (small groups are bound by latency), nothing in scratch memory."""
    k = kernels[f"group_wiener_kernel<{K}, {batch}, 0>"]
    assert waves_per_cu(k) >= 32 and k[".private_segment_fixed_size"] == 0
