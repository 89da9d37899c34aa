"""Registers and scratch of the built kernels, from the metadata of the library
(no GPU needed): the kernels of the default collision keep their values in
registers."""
import os
import re
import struct
import subprocess

import pytest

from paper_1908_05396_amd import build

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: scratch bytes per lane} of every kernel in libclbm.so."""
    with open(build.LIB, "rb") as fh:
        data = fh.read()
    out, at = {}, data.find(MAGIC)
    work = tmp_path_factory.mktemp("code")
    while at >= 0:
        p = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            p += 24 + idlen
            if size == 0 or data[at + off:at + off + 4] != b"\x7fELF":
                continue
            path = work / f"{at}_{off}.co"
            path.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
            for entry in notes.split("- .agpr_count:")[1:]:
                name = re.search(r"\.name:\s+(\S+)", entry)
                out[name.group(1)] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry).group(1))
        at = data.find(MAGIC, p)
    names = subprocess.run(["c++filt"], input="\n".join(out), check=True, capture_output=True, text=True).stdout
    return dict(zip(names.splitlines(), out.values()))


def _args(name):
    return re.search(r"<(.*?)>\(", name).group(1).split(", ")


def test_two_step_kernels_hold_their_values_in_registers(kernels):
    """Row layout, default collision without a force: no scratch in any storage
    type (the 12-row planes variant with its loads straight to LDS is apart)."""
    seen = 0
    for name, scratch in kernels.items():
        if "stream_collide2_kernel" not in name:
            continue
        _, _, forced, route, _, _, _, rows = _args(name)[:8]
        if rows == "true" and forced == "false" and route == "0":
            seen += 1
            assert scratch == 0, name
    assert seen >= 12
