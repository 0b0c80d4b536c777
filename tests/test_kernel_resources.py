"""Registers and scratch of the built kernels where a launch rule counts on them: read from the metadata of the library's own code
objects, no GPU needed."""
import os
import struct
import subprocess

import msgpack
import pytest

import paper_2604_10103_amd as hf


def _metadata(elf):
    """The AMDGPU metadata note of a 64-bit little-endian code object."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        at, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        end = at + size
        while kind == 7 and at < end:                     # SHT_NOTE
            name_len, desc_len, tag = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (name_len + 3) // 4 * 4
            if tag == 32:                                 # NT_AMDGPU_METADATA
                return msgpack.unpackb(elf[desc:desc + desc_len])
            at = desc + (desc_len + 3) // 4 * 4
    return {}


@pytest.fixture(scope="module")
def kernels():
    """Demangled name without arguments and namespaces -> the kernel's metadata."""
    with open(os.path.join(os.path.dirname(hf.__file__), "libhf.so"), "rb") as f:
        lib = f.read()
    found, at = {}, lib.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, = struct.unpack_from("<Q", lib, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, triple = struct.unpack_from("<QQQ", lib, p)
            if size and b"gfx950" in lib[p + 24:p + 24 + triple]:
                for k in _metadata(lib[at + off:at + off + size]).get("amdhsa.kernels", []):
                    found[k[".symbol"].removesuffix(".kd")] = k
            p += 24 + triple
        at = lib.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    plain = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.split("\n")
    tidy = lambda s: s.replace("(anonymous namespace)::", "").replace("hf::", "").removeprefix("void ").split("(")[0]
    return {tidy(name): k for name, k in zip(plain, found.values())}


@pytest.mark.parametrize("d", [64, 128])
def test_two_fp32_selecting_workgroups_share_a_compute_unit(kernels, d):
    """512 threads are two wavefronts a SIMD, of 512 registers."""
    assert kernels[f"pool_select_kernel<float, {d}>"][".vgpr_count"] <= 128


@pytest.mark.parametrize("instance,registers", [("bf16, 128, 1, 4, 4", 154), ("bf16, 64, 1, 4, 4", 84), ("float, 128, 1, 4, 4", 163),
                                                ("float, 64, 1, 4, 4", 99)])
def test_attention_without_selection_pays_nothing_for_it(kernels, instance, registers):
    """The instances for lists that are given share their source with the selecting ones: the counts from before they did."""
    name = f"attn_wide_kernel<{instance}, false>".replace("bf16", "unsigned short")
    assert kernels[name][".vgpr_count"] <= registers


@pytest.mark.parametrize("instance,spilled", [("2, 2, 0, 1", 4), ("4, 2, 0, 1", 3), ("8, 2, 0, 1", 3), ("2, 0, 1, 1", 7), ("2, 1, 1, 1", 9),
                                              ("2, 2, 1, 1", 16), ("4, 2, 1, 1", 3), ("2, 1, 1, 2", 0), ("4, 1, 1, 2", 0)])
def test_registers_that_the_bf16_attention_spills(kernels, instance, spilled):
    """Full launches of rotated queries and of selecting workgroups spill a few around their loop; nobody spills more."""
    assert kernels[f"attn_mfma_kernel<{instance}>"][".vgpr_spill_count"] <= spilled


def test_gradients_from_stored_scores_use_no_scratch(kernels):
    names = [n for n in kernels if n.startswith(("bwd_stored_kernel<", "bwd_scores_kernel<"))]
    assert len(names) == 24
    assert {n: kernels[n][".private_segment_fixed_size"] for n in names} == dict.fromkeys(names, 0)
