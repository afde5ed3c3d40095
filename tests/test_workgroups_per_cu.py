"""Narrow workgroups of the fused kernels per compute unit: as many as the LDS that the
selection needs allows, at every length that the host planner puts into such a launch.
Static LDS is what the built library's kernels declare; no GPU."""

import os
import shutil
import struct
import subprocess

import pytest

from launch_shapes import _driver
from paper_2503_08461_amd import fastcache

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
pytestmark = pytest.mark.skipif(not os.path.exists(READELF) or shutil.which("g++") is None, reason="no toolchain")

LDS, PIECE = 160 * 1024, 1280
VGPRS = 512  # of a SIMD; a narrow workgroup has one wavefront on each
KEEP = 16  # of the pruned kernel, next to what it shares with the selection


def kernels(tmp_path, details=None):
    """{mangled kernel name: (static LDS in bytes, vector registers)} of every kernel in the library;
    details: takes what else their descriptions say, {name: {key: count}}."""
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
            lds, more = None, {}
            for line in text.splitlines():
                key, _, value = line.strip().partition(":")
                if key == ".group_segment_fixed_size":
                    lds, more = int(value), {}
                elif key == ".symbol":
                    name = value.strip().removesuffix(".kd")
                elif key == ".vgpr_count":
                    out[name] = lds, int(value)
                if key in (".sgpr_count", ".vgpr_count", ".vgpr_spill_count") and details is not None:
                    more[key] = int(value)
                    if key == ".vgpr_spill_count":  # (the last)
                        details[name] = more
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


def test_pruned_kernels(tmp_path):
    built = kernels(tmp_path)
    select = built["_ZN2fc13select_kernelILi4EEEvNS_11BatchParamsE"][0]
    # the pruned form that the planner takes, for each number of query tiles (5: they differ)
    cases = [(d, tiles, L) for d in (64, 128) for tiles in (1, 2, 3, 4, 5) for L in range(512, 8193, 16)]
    text = ""
    for d, tiles, L in cases:
        more = "%d 1 %d 16\n" % (L, L // 5) if tiles == 5 else ""
        text += "1 600 %d 0 0 256 %d\n%d 1 %d %d\n%s" % (d, 2 if more else 1, L, L // 5, 16 * min(tiles, 4), more)
    out = subprocess.run([_driver()], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    launches = [[int(x) for x in line.split()[1:]] for line in out if line[0] == "F"]
    assert len(launches) == len(cases)
    for (wide, got_tiles, max_len, max_blocks, half, *_), (d, tiles, L) in zip(launches, cases):
        assert not wide and got_tiles == tiles and max_len == L
        name = "_ZN2fc20fused_bounded_kernelILi%dELi%dELi4ELb%dEEEvNS_11BatchParamsE"
        vgprs = built[name % (d, tiles, 0)][1]
        assert per_cu(*built[name % (d, tiles, half)], max_len, max_blocks) \
            == per_cu(select + KEEP, vgprs, max_len, max_blocks), (d, tiles, L, half)
        if d == 128 and L >= 2304:  # half of the keys are left to the caches wherever that costs no workgroup
            half_lds = built[name % (d, tiles, 1)][0]
            assert half == (per_cu(half_lds, vgprs, max_len, max_blocks) == per_cu(select + KEEP, vgprs, max_len, max_blocks))


def test_registers_grow_with_the_query_tiles(tmp_path):
    """A kernel for fewer query tiles needs no more registers than the next one (as it does where the
    compiler keeps an array of operands as one wide value)."""
    built = kernels(tmp_path)
    for family in ("17fused_unit_kernelILi%dELi%dELi4E", "19snapkv_score_kernelILi%dELi%dE",
                   "17split_rows_kernelILi%dELi%dE", "19split_scores_kernelILi%dELi%dE"):
        for d in (64, 128):
            vgprs = [built["_ZN2fc" + family % (d, tiles) + "EEvNS_11BatchParamsE"][1] for tiles in (1, 2, 3, 4)]
            assert vgprs == sorted(vgprs), (family, d, vgprs)


def test_vector_spills(tmp_path):
    """The pruned kernels of four and of mixed query tiles, which fill the registers, spill no more
    than a head writes and reads back a few times; no other kernel of the scores spills at all."""
    details = {}
    kernels(tmp_path, details)
    spilling = {name: x[".vgpr_spill_count"] for name, x in details.items() if x[".vgpr_spill_count"] and "mlp" not in name}
    assert all("fused_bounded" in name and ("ELi4ELi" in name or "ELi5ELi" in name) for name in spilling), spilling
    assert max(spilling.values()) <= 9, spilling


def test_wavefronts_per_simd(tmp_path):
    """Heads so short that LDS does not limit them: what the registers of the kernels that score in
    full allow, and two wide workgroups a CU at 64 channels with at most one query tile."""
    details = {}
    kernels(tmp_path, details)

    def wavefronts(name):
        x = details["_ZN2fc%sEEvNS_11BatchParamsE" % name]
        # (a SIMD has 800 scalar registers; 16 of each wavefront are the trap handler's)
        return min(VGPRS // (-(-x[".vgpr_count"] // 8) * 8), 800 // (-(-(x[".sgpr_count"] + 16) // 16) * 16))
    least = {(128, 0): 5, (128, 1): 5, (128, 2): 4, (128, 3): 4, (128, 4): 3, (128, 5): 3,
             (64, 0): 7, (64, 1): 8, (64, 2): 7, (64, 3): 5, (64, 4): 4, (64, 5): 4}
    for (d, tiles), n in least.items():
        assert wavefronts("17fused_unit_kernelILi%dELi%dELi4E" % (d, tiles)) >= n, (d, tiles)
    for name in ("17fused_unit_kernelILi64ELi0ELi16E", "17fused_unit_kernelILi64ELi1ELi16E", "22fused_unit_only_kernelILi64ELi16E",
                 "20fused_bounded_kernelILi64ELi1ELi16ELb0E", "25fused_bounded_only_kernelILi64ELi1ELi16E"):
        assert wavefronts(name) == 8, name


def test_kernel_names_of_the_benchmark(tmp_path):
    """The names that the benchmark prints are kernels of the library, the one with half of the
    keys left to the caches where the planner takes it."""
    import re
    import bench
    from paper_2503_08461_amd import synth
    built = kernels(tmp_path)
    for config, pruning in [(1, True), (2, True), (2, False), (3, True), (4, True), (4, False), (5, True)]:
        wl = synth.make_workload(config)
        name = bench.kernel_symbol("fused_unit", wl, pruning)
        kernel, args = re.fullmatch(r"fc::(\w+)<(.*)>", name).groups()
        args = ["Lb%d" % (a == "true") if a in ("true", "false") else "Li" + a for a in args.split(", ")]
        assert "_ZN2fc%d%sI%sEEvNS_11BatchParamsE" % (len(kernel), kernel, "E".join(args) + "E") in built, name
        if pruning:
            text = "%d %d %d 0 0 256 %d\n" % (wl.n_layers, wl.n_heads, wl.head_dim, wl.n_req) + "".join(
                "%d %d %d %d\n" % r for r in zip(wl.seq_lens, wl.methods, wl.budgets, [wl.window] * wl.n_req))
            out = subprocess.run([_driver()], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
            assert any(int(line.split()[5]) for line in out if line[0] == "F") == name.endswith("true>"), name
            one = subprocess.run([_driver(), "one"], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
            assert int(one[0].split()[1]) == ("_only_kernel<" in name), name
            launches = [line.split() for line in out if line[0] == "F" and kernel.startswith("fused")]
            assert any((w != "0") == (args[2] != "Li4") for _, w, *_ in launches), name
