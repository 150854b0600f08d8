"""Registers of the built kernels: waves per SIMD and spills that the launch rules and the kernels' layout were measured with.

Read from the metadata notes of the code objects inside the built library, so no GPU is needed."""
import re
import struct
import subprocess
from pathlib import Path

import pytest

from paper_2406_09827_amd import build

LLVM = Path(build.HIPCC).resolve().parents[1] / "llvm" / "bin"


def _code_objects(library: bytes):
    """The gfx950 code objects of every offload bundle (one per translation unit)."""
    at = 0
    while (at := library.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", library, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", library, entry)
            if library[entry + 24:entry + 24 + length].endswith(b"gfx950") and size:
                yield library[at + offset:at + offset + size]
            entry += 24 + length
        at += 24


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel with its template arguments: {"waves": per SIMD by registers, "spilled": vector registers}}"""
    if not Path(build.LIB).exists():
        build.build_lib()
    found = {}
    for i, code in enumerate(_code_objects(Path(build.LIB).read_bytes())):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(code)
        notes = subprocess.run([str(LLVM / "llvm-readelf"), "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for part in notes.split(".agpr_count:")[1:]:
            number = {k: int(v) for k, v in re.findall(r"\.(vgpr_count|vgpr_spill_count): +(\d+)", part)}
            found[re.search(r"\.symbol: +'?(\S+?)\.kd", part)[1]] = dict(waves=min(8, 512 // (-(-number["vgpr_count"] // 8) * 8)), spilled=number["vgpr_spill_count"])
    names = subprocess.run(["c++filt"], input="\n".join(found), check=True, capture_output=True, text=True).stdout.split("\n")
    table = {re.sub(r"^void |hipattn::|\(anonymous namespace\)::|\(.*$| ", "", n.replace("(anonymous namespace)::", "")): v for n, v in zip(names, found.values())}
    assert len(table) > 600
    return table


def check(kernels, waves, spilled, name):
    got = kernels[name]
    assert got["waves"] >= waves and got["spilled"] <= spilled, (name, got)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [1, 2, 4, 8])
def test_decode_mask_of_few_nodes_runs_five_waves(kernels, rows, d):
    # one wave a problem: contiguous and paged; four: contiguous (128 channels with two or four rows a block: four waves)
    for mode in (0, 1):
        check(kernels, 5, 0, f"mask_decode_kernel<2,{rows},{d},8,{mode},1>")
    four = d == 128 and rows in (2, 4)
    for mode in (0, 2):
        check(kernels, 4 if four else 5, 0 if four else 1, f"mask_decode_kernel<2,{rows},{d},8,{mode},4>")
    check(kernels, 4, 0, f"mask_decode_kernel<2,{rows},{d},8,1,4>")
