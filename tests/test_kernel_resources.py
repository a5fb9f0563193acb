"""Registers of the compiled kernels, from the metadata in the built library: the prompt GEMMs that the plan can take keep
their state in registers."""
import struct
import subprocess

import msgpack
import pytest

import paper_2410_01028_amd as asd


def kernels():
    """Metadata of the gfx950 kernels in the library, by demangled name."""
    lib = open(asd.LIB_PATH, "rb").read()
    start = lib.index(b"__CLANG_OFFLOAD_BUNDLE__")
    at, elf = start + 32, None
    for _ in range(struct.unpack_from("<Q", lib, start + 24)[0]):
        offset, size, n = struct.unpack_from("<QQQ", lib, at)
        if b"gfx950" in lib[at + 24:at + 24 + n]:
            elf = lib[start + offset:start + offset + size]
        at += 24 + n
    sections, = struct.unpack_from("<Q", elf, 40)
    each, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * each + 4)
        at, size = struct.unpack_from("<QQ", elf, sections + i * each + 24)
        end = at + size
        while kind == 7 and at < end:                                     # SHT_NOTE
            n_name, n_desc, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (n_name + 3) // 4 * 4
            if note == 32 and elf[at + 12:at + 18] == b"AMDGPU":           # NT_AMDGPU_METADATA
                found = msgpack.unpackb(elf[desc:desc + n_desc])["amdhsa.kernels"]
                names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True, check=True).stdout.splitlines()
                return dict(zip((n.split("(")[0].removeprefix("void ") for n in names), found))
            at = desc + (n_desc + 3) // 4 * 4
    raise AssertionError("no kernel metadata")


@pytest.fixture(scope="module")
def table():
    return kernels()


def spills(table, prefix):
    chosen = {n: k for n, k in table.items() if n.startswith(prefix)}
    assert chosen
    return {n: (k[".sgpr_spill_count"], k[".vgpr_spill_count"]) for n, k in chosen.items() if k[".sgpr_spill_count"] or k[".vgpr_spill_count"]}


@pytest.mark.parametrize("epilogue", [1, 2], ids=["raw", "gate/up"])
@pytest.mark.parametrize("dtype", ["BF16", "F32"])
def test_ring_kernel_spills_nothing(table, dtype, epilogue):
    assert spills(table, f"pf_ring_kernel<{dtype}, {epilogue},") == {}


@pytest.mark.parametrize("dtype", ["BF16", "F32"])
def test_qkv_epilogue_spills_nothing(table, dtype):
    assert spills(table, f"pf_ring_kernel<{dtype}, 0,") == {}
    four_wave = spills(table, f"pf_gemm_kernel<{dtype}, 0,")
    # eight chunks fill the registers of the bf16 kernel's main loop (the raw sums' spills as many vector registers), nothing else does
    full = spills(table, f"pf_gemm_kernel<{dtype}, 1,").get(f"pf_gemm_kernel<{dtype}, 1, 4, 8, 4, 2>", (0, 0))
    assert {n: s for n, s in four_wave.items() if "4, 8, 4, 2>" not in n} == {}
    assert four_wave.get(f"pf_gemm_kernel<{dtype}, 0, 4, 8, 4, 2>", (0, 0)) <= full
