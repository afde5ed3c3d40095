"""Narrow workgroups of the fused kernels per compute unit: as many as the LDS that the
selection needs allows, at every length that the host planner puts into such a launch.
Static LDS is what the built library's kernels declare; no GPU."""

import os
import struct
import subprocess

import pytest

from paper_2503_08461_amd import fastcache

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
pytestmark = pytest.mark.skipif(not os.path.exists(READELF), reason="no toolchain")

LDS, PIECE = 160 * 1024, 1280
VGPRS = 512  # of a SIMD; a narrow workgroup has one wavefront on each


def kernels(tmp_path):
    """{mangled kernel name: (static LDS in bytes, vector registers)} of every kernel in the library."""
    lib = open(fastcache.LIB_PATH, "rb").read()
    out, at = {}, lib.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", lib, at + 18)[0] == 224:  # a code object for the GPU
            # (section headers come last)
            end = at + struct.unpack_from("<Q", lib, at + 40)[0] + \
                struct.unpack_from("<H", lib, at + 58)[0] * struct.unpack_from("<H", lib, at + 60)[0]
            path = tmp_path / "code"
            path.write_bytes(lib[at:end])
            text = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            lds = None
            for line in text.splitlines():
                key, _, value = line.strip().partition(":")
                if key == ".group_segment_fixed_size":
                    lds = int(value)
                elif key == ".symbol":
                    name = value.strip().removesuffix(".kd")
                elif key == ".vgpr_count":
                    out[name] = lds, int(value)
        at = lib.find(b"\x7fELF", at + 4)
    return out


def per_cu(static, vgprs, max_len, max_blocks):
    """Workgroups whose scores, token bits and block ids lie behind `static` bytes."""
    words = 4 + (max_len + 3) // 4 * 4 + 8 + (max_len + 255) // 256 * 8 + (min(max_blocks, 512) + 3) // 4 * 4
    return min(LDS // (-(-(static + 4 * words) // PIECE) * PIECE), VGPRS // (-(-vgprs // 8) * 8), 8)


def test_kernels_that_score_in_full(tmp_path):
    built = kernels(tmp_path)
    select = built["_ZN2fc13select_kernelILi4EEEvNS_11BatchParamsE"][0]
    for d in (64, 128):
        for tiles in range(6):
            lds, vgprs = built["_ZN2fc17fused_unit_kernelILi%dELi%dELi4EEEvNS_11BatchParamsE" % (d, tiles)]
            for L in range(16, 8193, 16):
                assert per_cu(lds, vgprs, L, L // 16) == per_cu(select, vgprs, L, L // 16), (d, tiles, L)
