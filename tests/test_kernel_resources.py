"""Host only: what the compiler gave each kernel of the built library, read from the metadata that
the code objects carry (registers, scratch, static LDS)."""
import re
import struct
import subprocess

import msgpack
import pytest

import paper_2408_07092_amd as ds

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects of a library: entries of its uncompressed offload bundles."""
    data = open(path, "rb").read()
    for m in re.finditer(re.escape(BUNDLE), data):
        base, pos = m.start(), m.start() + len(BUNDLE) + 8
        for _ in range(struct.unpack_from("<Q", data, base + len(BUNDLE))[0]):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + n].decode()
            pos += 24 + n
            if "gfx950" in name:
                yield data[base + off:base + off + size]


def kernel_metadata(elf):
    """amdhsa.kernels of a code object: the msgpack note of type 32 in its note segments."""
    assert elf[:4] == b"\x7fELF"
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
        if kind != 4:  # PT_NOTE
            continue
        pos, end = off, off + size
        while pos + 12 <= end:
            n_name, n_desc, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (n_name + 3) // 4 * 4
            if note == 32:
                return msgpack.unpackb(elf[desc:desc + n_desc], strict_map_key=False)["amdhsa.kernels"]
            pos = desc + (n_desc + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def kernels():
    ds.lib()  # (raises if the library has not been built)
    found = [k for elf in code_objects(ds.binding.LIB_PATH) for k in kernel_metadata(elf)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True,
                           text=True, check=True).stdout.splitlines()
    out = {re.sub(r"^void ", "", n).split("(")[0].removeprefix("ds::"): k for n, k in zip(names, found)}
    assert len(out) == len(found) > 40 and "k_attend<1, 1>" in out
    return out


def test_no_kernel_uses_scratch_memory(kernels):
    """Every kernel's registers fit the occupancy that its launch bounds ask for: nothing is spilled
    to scratch memory."""
    spilled = {n: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for n, k in kernels.items()
               if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not spilled


def test_q4_build_is_limited_by_its_tile_alone(kernels):
    """What make_q4_plan counts on: eight workgroups to a compute unit by registers, and no more static
    LDS than it allows for."""
    k = kernels["k_q4_build"]
    assert k[".vgpr_count"] + k.get(".agpr_count", 0) <= 64 and k[".group_segment_fixed_size"] <= 1280


def test_k_row_scoring_keeps_its_loads_in_flight(kernels):
    """32 loads of a lane at once, with or without the bins: more registers than the compiler would give them if
    it aimed at eight wavefronts to a SIMD, and few enough for four."""
    found = {n: k[".vgpr_count"] + k.get(".agpr_count", 0) for n, k in kernels.items() if "k_scoreILin2ELb" in n}
    assert len(found) == 2 and all(64 < v <= 104 for v in found.values()), found


def test_decode_kernels_leave_room_for_the_workgroups_that_plans_count_on(kernels):
    """Four wavefronts to a SIMD (128 registers), two workgroups of 512 threads or four of 256 to a compute unit;
    for groups of more than eight heads three (168)."""
    seen = 0
    for n, k in kernels.items():
        m = re.match(r"k_refine_attend<(\d+), (-?\d+), (\d+), (true|false)>", n)
        if m:
            seen += 1
            assert k[".vgpr_count"] + k.get(".agpr_count", 0) <= (128 if int(m.group(1)) <= 8 else 168), n
    assert seen == 11 * (2 * 4 + 3 * 2)  # (label sources; forms of single heads and pairs, of groups)
