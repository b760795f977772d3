"""Static LDS of the kernels whose dynamic LDS is sized to a share of a CU.

k_tile_scatter's default tiles take exactly a quarter of a CU's LDS at some
column counts, so a single static word takes a whole block off every CU.  The
sizes are read from the metadata of the built library.
"""
import os
import struct
import subprocess

import pytest
import yaml

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2509_14433_amd", "libcupk.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 code objects of every offload bundle in a host library."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24: p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off: at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def test_tile_scatter_has_no_static_lds(tmp_path):
    if not (os.path.exists(LIB) and os.path.exists(READELF)):
        pytest.skip("no built library or no llvm-readelf")
    with open(LIB, "rb") as f:
        data = f.read()
    lds = {}
    for i, obj in enumerate(_code_objects(data)):
        path = tmp_path / f"{i}.o"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        meta = yaml.safe_load(notes[notes.index("---"):].split("\n...")[0])
        for k in meta["amdhsa.kernels"]:
            lds[k[".symbol"]] = k[".group_segment_fixed_size"]
    tiles = {k: v for k, v in lds.items() if "14k_tile_scatter" in k or "19k_tile_scatter_stag" in k}
    assert len(tiles) >= 3, sorted(lds)
    assert all(v == 0 for v in tiles.values()), tiles
