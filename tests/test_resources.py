"""What the launch rules assume of the kernels' resources, held against the built library (CPU only: the resources are read from
the notes of the code objects that this repository's own build has put into it)."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_25463_amd", "csrc")
LLVM = "/opt/rocm/llvm/bin"
UNIT_LDS, LDS_GRANULE, REGISTERS = 160 * 1024, 1280, 512           # of a compute unit; per lane of a SIMD


def code_objects(lib, tmp):
    """The gfx950 code objects of the library's offload bundles."""
    fat = str(tmp / "fatbin")
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, lib, str(tmp / "copy")], check=True)
    data = open(fat, "rb").read()
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.end() + 8
        for _ in range(struct.unpack_from("<Q", data, m.end())[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            if b"gfx950" in data[at + 24:at + 24 + name]:
                yield data[m.start() + offset:m.start() + offset + size]
            at += 24 + name


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{'stream_kernel<bf16_t, 64, 8, ...>': dict(lds=, scratch=, registers=)} of every kernel in the library."""
    from paper_2603_25463_amd import build
    build.build(force=False)
    tmp = tmp_path_factory.mktemp("code")
    found = {}
    for i, obj in enumerate(code_objects(build.LIB, tmp)):
        path = tmp / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for note in notes.split("  - .agpr_count")[1:]:
            field = lambda name: re.search(r"\.%s:\s*(\S+)" % name, note)[1]
            mangled = re.search(r"\s\.name:\s*(_Z\S+)", note)[1]
            found[mangled] = dict(lds=int(field("group_segment_fixed_size")), scratch=int(field("private_segment_fixed_size")),
                                  registers=int(field("vgpr_count")))
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.splitlines()
    short = [re.sub(r"^void |ciar::|\(anonymous namespace\)::", "", n).split("(")[0] for n in names]
    return dict(zip(short, found.values()))


def fits(k, threads, dynamic):
    """Workgroups of a kernel that a compute unit has room for."""
    lds = -(-(k["lds"] + dynamic) // LDS_GRANULE) * LDS_GRANULE
    waves = 4 * (REGISTERS // (-(-k["registers"] // 8) * 8))
    return min(UNIT_LDS // max(lds, 1), waves * 64 // threads, 2048 // threads)


def test_the_grids_count_on_no_more_workgroups_than_a_compute_unit_has_room_for(kernels, tmp_path):
    """A grid of a round more workgroups than are resident ends in a nearly empty round (whole_rounds is there to prevent it)."""
    lines = ['#include "ciar_stream.h"', '#include "ciar_loss.hip"', "using namespace ciar;"]
    for name, k in kernels.items():
        kernel, args = re.fullmatch(r"(\w+)(?:<(.*)>)?", name).groups()
        if kernel == "stream_kernel":
            a = args.split(", ")
            through_lds = f"next_by_lds<{a[0]}, {a[1]}, {a[2]}, {a[4]}, {a[5]}, {a[6]}>()"
            dynamic, threads, asked = int(a[1]) * int(a[2]) * 16, int(a[1]), f"workgroups_per_unit<{', '.join(a[:7])}>()"
            room = f"({through_lds} ? {fits(k, threads, dynamic)} : {fits(k, threads, 0)})"
        elif kernel == "dro_row_stream_kernel":
            a = args.split(", ")
            dynamic, threads, asked = 2 * int(a[1]) * int(a[2]) * 16, int(a[2]), f"dro_workgroups_per_unit<{args}>()"
            room = str(fits(k, threads, dynamic))
        else:
            continue
        lines.append(f'static_assert({asked} <= {room}, "{name}");')
    assert len(lines) > 100
    source = tmp_path / "held.hip"
    source.write_text("\n".join(lines) + "\n")
    r = subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only", "-std=c++17", "-w",
                        "-I", CSRC, str(source)], capture_output=True, text=True)
    assert r.returncode == 0, "\n".join(l for l in r.stderr.splitlines() if "error" in l)


def test_rows_that_come_through_lds_are_not_waited_for_by_a_scratch_reload(kernels):
    """A reload of a spilled register waits for every load in flight, the next row's among them."""
    persistent = {n: k["scratch"] for n, k in kernels.items() if n.startswith("dro_row_stream_kernel") and n.endswith("false>")}
    assert len(persistent) >= 10 and not any(persistent.values()), persistent
