"""Resources of the built kernels, as the library's own code objects state them (no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2410_03355_amd as lantern

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
READELF, OBJDUMP = os.path.join(LLVM, "llvm-readelf"), os.path.join(LLVM, "llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_objects(blob):
    """gfx950 code objects of every offload bundle in the library: after the magic the number of entries, then per
    entry its offset from the magic, its size, and the length and text of its target."""
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in target and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + len(MAGIC))


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """Paths of the library's code objects, each in a file of its own."""
    if not os.path.exists(lantern.LIB_PATH):
        lantern.build()
    with open(lantern.LIB_PATH, "rb") as f:
        blob = f.read()
    paths = []
    for i, obj in enumerate(_device_objects(blob)):
        paths.append(tmp_path_factory.mktemp("objects") / f"{i}.o")
        paths[-1].write_bytes(obj)
    return paths


@pytest.fixture(scope="module")
def kernels(objects):
    """{mangled name: (bytes of scratch per lane, spilled vector registers, vector registers, bytes of LDS fixed at
    compile time)}"""
    found = {}
    for path in objects:
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for part in notes.split("- .agpr_count")[1:]:
            value = {key: re.search(r"\." + key + r":\s+(\S+)", part).group(1)
                     for key in ("name", "private_segment_fixed_size", "vgpr_spill_count", "vgpr_count",
                                 "group_segment_fixed_size")}
            found[value["name"]] = (int(value["private_segment_fixed_size"]), int(value["vgpr_spill_count"]),
                                    int(value["vgpr_count"]), int(value["group_segment_fixed_size"]))
    assert len(found) > 50
    return found


def test_sequential_walk_keeps_out_of_scratch(kernels):
    """The walk under total variation (template arguments: logit type, steps, plain rule, divergence)."""
    walks = {name: r for name, r in kernels.items() if re.search(r"trees_sequentialI[ft]Li\d+ELb0ELb0EE", name)}
    assert len(walks) == 8
    for name, (scratch, spilled, *_) in walks.items():
        steps = int(re.search(r"Li(\d+)E", name).group(1))
        assert (scratch, spilled) <= ((8, 1) if steps == 10 else (0, 0)), name


def test_smallest_full_rows_leave_room_for_five_wavefronts(kernels):
    """The fp32 pass over fp32 rows of 4 KiB (256 threads, one vector, full rows, vector table): up to 96 registers
    five wavefronts fit a SIMD, and 30720 such rows take 87 us instead of 104."""
    name, = [n for n in kernels if re.search(r"verify_fastIfLi256ELi1ELi0ELb1EE", n)]
    assert kernels[name][0] == 0 and kernels[name][2] <= 96


def test_selections_from_whole_rows_by_elements(kernels):
    """Whole rows of any number of keys have a selection that reads codes element by element (last template argument) and holds
    nothing of the vectors' way: fewer registers, no scratch."""
    for code in "ft":
        for keys, threads, most in ((0, 256, (48, 62)), (8, 256, (48, 62)), (32, 256, (64, 64)), (64, 256, (128, 128)), (64, 512, (128, 128))):
            for slots, limit in zip((256, 1024), most):
                name, = [n for n in kernels if re.search(rf"knn_selectI{code}Li{keys}ELi{slots}ELi{threads}ELb0ELi0EE", n)]
                assert kernels[name][0] == 0 and kernels[name][2] <= limit, name


def test_rows_arrive_without_scratch_memory(objects):
    """Until a row is in LDS (the first barrier) no kernel of the fp32 pass touches scratch memory."""
    seen = 0
    for path in objects:
        listing = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                                 check=True, capture_output=True, text=True).stdout
        for name, body in re.findall(r"^<(\S*verify_fast\S*)>:\n(.*?)(?=^<|\Z)", listing, re.S | re.M):
            arriving = body[:body.index("s_barrier")]
            assert "global_load_dwordx4" in arriving and "scratch_" not in arriving, name
            seen += 1
    assert seen == 42


def test_exponential_tables_are_objects_of_their_own(kernels):
    """The 4 KiB table of the fp64 exponential has a place in LDS that the compiler gives it and knows, wherever that is: no
    lookup goes to an absolute address."""
    assert all(r[3] >= 4096 for n, r in kernels.items() if re.search("verify_fast|trees_sequential", n))
    csrc = os.path.join(os.path.dirname(lantern.LIB_PATH), "csrc")
    for name in os.listdir(csrc):
        with open(os.path.join(csrc, name)) as f:
            assert "address_space(3)" not in f.read(), name


def test_filtering_contraction_keeps_out_of_scratch(kernels):
    """Every form of it (key, list, tokens to a tile): setting up scratch memory alone is felt in launches of this length."""
    filters = {name: r for name, r in kernels.items() if "knn_filter_list" in name}
    assert len(filters) == 12
    for name, r in filters.items():
        assert r[:2] == (0, 0), name
