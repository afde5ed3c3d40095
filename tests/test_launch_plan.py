"""How a compress call's heads are spread over workgroups (csrc/fc_plan.cpp):
every unit in exactly one launch, heads within the launch's limits, the sizes at
which the shapes change, and offsets of split heads.  Host code, built with the
sanitizers, no GPU."""

import os
import random
import shutil
import subprocess

import pytest

from conftest import ROOT

SNAP, KNORM, STREAM = 1, 2, 3
N_CU = 256


def _case(nl, nh, reqs, mode=0, in_place=0, d=128, n_cu=N_CU):
    return (nl, nh, d, mode, in_place, n_cu, reqs)


def _random_case(rng):
    nl, nh = rng.choice([(1, 4), (1, 32), (2, 32), (32, 32)])
    reqs = []
    for _ in range(rng.randrange(1, 40)):
        m = rng.choice([SNAP, SNAP, KNORM, STREAM])
        w = rng.randrange(1, 65)
        L = max(w, int(2 ** rng.uniform(0, 15)))
        reqs.append((L, m, rng.randrange(w, L + 1) if m == SNAP else rng.randrange(1, L + 1), w))
    return _case(nl, nh, reqs, rng.choice([0, 0, 0, 1]), rng.choice([0, 0, 1]))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_launch_plan(tmp_path):
    exe = str(tmp_path / "launch_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", os.path.join(ROOT, "tests", "launch_plan_driver.cpp"),
                    os.path.join(ROOT, "paper_2503_08461_amd", "csrc", "fc_plan.cpp"), "-o", exe], check=True)
    long1 = [(2048, SNAP, 400, 32)]
    edges = [
        (_case(1, 128, long1), "split"),                 # one head per two compute units
        (_case(1, 129, long1), "wide"),
        (_case(1, 128, [(2047, SNAP, 400, 32)], d=64), "wide"),  # too short to split
        (_case(1, 128, long1, in_place=1), "wide"),      # one workgroup per head copies in place
        (_case(1, 256, long1), "wide"),
        (_case(1, 257, long1), "narrow"),                # a second round
        (_case(1, 513, [(8192, SNAP, 400, 32)]), "narrow"),
        (_case(1, 513, [(8193, SNAP, 400, 32)]), "wide"),
        # one round of wide workgroups at most, from the length on that keeps them busy
        (_case(1, 256, [(2047, SNAP, 100, 32)]), "narrow"),
        (_case(1, 256, [(2048, SNAP, 100, 32)]), "wide"),
        (_case(1, 256, [(895, SNAP, 100, 32)], d=64), "narrow"),
        (_case(1, 256, [(896, SNAP, 100, 32)], d=64), "wide"),
        (_case(1, 257, [(8000, SNAP, 100, 32)], d=64), "narrow"),
        (_case(1, 256, [(255, KNORM, 100, 32)]), "narrow"),
        (_case(1, 256, [(256, KNORM, 100, 32)]), "wide"),
        (_case(1, 257, [(8000, KNORM, 100, 32)]), "narrow"),
        (_case(1, 256, [(255, STREAM, 100, 32)]), "narrow"),
        (_case(1, 256, [(256, STREAM, 100, 32)]), "wide"),
        (_case(1, 128, [(4000, SNAP, 1000, 32)] + [(2000, SNAP, 500, 32)] * 2), "wide"),   # as much as 256 of the first
        (_case(1, 128, [(4000, SNAP, 1000, 32)] + [(2001, SNAP, 500, 32)] * 2), "narrow"),
        (_case(1, 128, [(1000, SNAP, 200, 32), (1000, KNORM, 200, 32)]), "narrow"),        # the heaviest decides
        (_case(1, 128, [(1000, SNAP, 200, 32), (4000, KNORM, 200, 32)]), "wide"),
        (_case(1, 4, [(256, SNAP, 64, 16)]), "narrow"),
        (_case(1, 32, [(100, SNAP, 64, 16), (9, KNORM, 4, 16), (20000, STREAM, 4000, 16)]), "wide"),
    ]
    rng = random.Random(7)
    cases = [c for c, _ in edges] + [_random_case(rng) for _ in range(300)]
    text = "".join("%d %d %d %d %d %d %d\n%s\n" % (c[:6] + (len(c[6]), "\n".join("%d %d %d %d" % r for r in c[6])))
                   for c in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    parsed = []
    for line in out.splitlines():
        row = [int(x) for x in line.split()[1:]]
        if line[0] == "C":
            parsed.append((row, []))
        elif line[0] == "F":
            parsed[-1][1].append(row)
    assert len(parsed) == len(cases)
    for (head, launches), (_, want) in zip(parsed, edges):
        got = "split" if head[0] else "wide" if launches[0][0] else "narrow"
        assert got == want and len(launches) == 1
    n_split = 0
    for ((split, raw_floats, *raw_offs), launches), (nl, nh, _, mode, in_place, n_cu, reqs) in zip(parsed, cases):
        units = nl * nh
        if split:
            n_split += 1
            assert mode == 0 and not in_place and units * len(reqs) <= n_cu // 2
            at = 0
            for (L, *_), off in zip(reqs, raw_offs):
                assert off == at
                at += units * L
            assert raw_floats == at and 2 <= split <= max(L for L, m, *_ in reqs if m != STREAM) // 256
        seen = []
        for wide, tiles, max_len, max_blocks, _, *members in launches:
            seen += members
            lens = [reqs[i][0] for i in members]
            scored = [reqs[i][0] for i in members if reqs[i][1] != STREAM]
            classes = {(reqs[i][3] + 15) // 16 for i in members if reqs[i][1] == SNAP}
            assert max_len == max(scored, default=0) <= (32768 if wide else 8192)
            assert max_blocks == max((L + 15) // 16 for L in lens)
            assert tiles == (0 if not classes else 5 if len(classes) > 1 else classes.pop())
            weight = [2 * reqs[i][0] * (reqs[i][1] == SNAP) + reqs[i][0] * (reqs[i][1] == KNORM) + 4 * reqs[i][2]
                      for i in members]
            assert weight == sorted(weight, reverse=True)
        # (with the separate scheduling only streaming requests run in the fused kernels)
        assert sorted(seen) == [i for i, r in enumerate(reqs) if mode == 0 or r[1] == STREAM]
        assert len(launches) <= 2
    assert n_split > 5


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_which_launches_leave_half_of_the_keys_to_the_caches():
    """Narrow workgroups at 128 channels from a mean length of their SnapKV heads (weighted by
    itself) on, unless the kernel that does it would cost a CU a workgroup."""
    from launch_shapes import _driver

    def snap(*lens, w=32):
        return [(L, SNAP, max(w, L // 5), w) for L in lens]
    fillers = [(9, KNORM, 4, 32)] * 600
    cases = [
        (_case(1, 600, snap(2303)), 0),
        (_case(1, 600, snap(2304)), 1),
        (_case(1, 256, snap(8000)), 0),                      # wide
        (_case(1, 600, snap(8000), d=64), 0),
        (_case(1, 1, snap(2303, 2303) + fillers), 0),        # other methods do not count
        (_case(1, 1, snap(2304, 2304) + fillers), 1),
        (_case(1, 600, [(8000, KNORM, 400, 32)] + snap(2303)), 0),
        (_case(1, 600, snap(1000, 3000)), 1),                # (1000^2 + 3000^2) / 4000 = 2500
        (_case(1, 600, snap(1000, 1000, 3000)), 0),          # 2200
        (_case(1, 600, snap(8192)), 1),
        (_case(1, 600, snap(7820, w=48)), 1),
        (_case(1, 600, snap(7821, w=48)), 0),
        (_case(1, 600, snap(7821, w=32) + snap(3000, w=16)), 0),   # two classes of windows
        (_case(1, 600, snap(7820, w=32) + snap(3000, w=16)), 1),
        (_case(1, 600, [(7821, KNORM, 400, 32)] + snap(3000, w=64)), 0),
        (_case(1, 600, [(20000, STREAM, 400, 32)] + snap(7800, w=64)), 1),  # a longer table of block ids
        (_case(1, 600, [(20000, STREAM, 400, 32)] + snap(7801, w=64)), 0),
    ]
    text = "".join("%d %d %d %d %d %d %d\n%s\n" % (c[:6] + (len(c[6]), "\n".join("%d %d %d %d" % r for r in c[6])))
                   for c, _ in cases)
    out = subprocess.run([_driver()], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    got = [[int(x) for x in line.split()[1:]] for line in out if line[0] == "F"]
    assert [launch[4] for launch in got] == [want for _, want in cases]


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_which_calls_go_without_plan_alloc():
    """One request in one fused launch, as a pruned call and as one that is not: up to 512 block
    ids and a million tokens of all heads; many heads only where they are long enough not to
    come to the counter all at once."""
    from launch_shapes import _driver
    cases = [
        (_case(1, 4, [(256, SNAP, 64, 16)], d=64), (1, 0)),
        (_case(1, 4, [(256, KNORM, 64, 16)], d=64), (1, 1)),
        (_case(1, 4, [(256, STREAM, 64, 16)], d=64), (0, 0)),
        (_case(1, 4, [(256, SNAP, 64, 16)], mode=1), (0, 0)),
        (_case(1, 4, [(256, KNORM, 64, 16)], mode=1), (0, 0)),
        (_case(1, 4, [(256, STREAM, 64, 16)], mode=1), (0, 0)),
        (_case(1, 4, [(256, SNAP, 64, 16)] * 2), (0, 0)),
        (_case(1, 128, [(2047, SNAP, 400, 32)]), (1, 0)),
        (_case(1, 128, [(2048, SNAP, 400, 32)]), (0, 0)),            # split
        (_case(1, 128, [(2048, SNAP, 400, 32)], in_place=1), (1, 0)),
        (_case(1, 136, [(6000, SNAP, 2192, 16)], d=64), (1, 0)),     # 375 + 137 ids
        (_case(1, 136, [(6000, SNAP, 2193, 16)], d=64), (0, 0)),
        (_case(1, 136, [(6000, SNAP, 6000, 16)], d=64, in_place=1), (1, 0)),  # (no new ones)
        (_case(32, 32, [(1024, SNAP, 200, 32)]), (1, 0)),            # 1 << 20 tokens
        (_case(32, 32, [(1025, SNAP, 200, 32)]), (0, 0)),
        # more than 256 heads: from 400 tokens of 128 channels on
        (_case(8, 32, [(20, KNORM, 9, 32)]), (1, 1)),
        (_case(1, 257, [(399, KNORM, 100, 32)]), (0, 0)),
        (_case(1, 257, [(400, KNORM, 100, 32)]), (1, 1)),
        (_case(1, 257, [(799, SNAP, 100, 32)], d=64), (0, 0)),
        (_case(1, 257, [(800, SNAP, 100, 32)], d=64), (1, 0)),
        (_case(32, 32, [(300, KNORM, 90, 32)], d=64), (0, 0)),
    ]
    text = "".join("%d %d %d %d %d %d %d\n%s\n" % (c[:6] + (len(c[6]), "\n".join("%d %d %d %d" % r for r in c[6])))
                   for c, _ in cases)
    out = subprocess.run([_driver(), "one"], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    for (case, want), line in zip(cases, out):
        assert tuple(int(x) for x in line.split()[1:]) == want, (case, line)
    assert len(out) == len(cases)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_lengths_from_which_heads_are_pruned():
    """Longer with more query tiles, in wide workgroups and with fewer heads; never so short that a
    head's first step reaches its window (64 tokens a narrow workgroup, 256 a wide one)."""
    from launch_shapes import _driver
    cases = [_case(1, heads, [(L, SNAP, 100, 32)], d=d) for d in (64, 128) for heads, L in
             ((513, 8192), (512, 8192), (256, 200), (256, 8192))]
    text = "".join("%d %d %d %d %d %d %d\n%s\n" % (c[:6] + (1, "%d %d %d %d" % c[6][0])) for c in cases)
    out = subprocess.run([_driver()], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    limits = [[int(x) for x in line.split()[1:]] for line in out if line[0] == "P"]
    assert [line[2] for line in out if line[0] == "F"] == list("00010001")
    for d, (many, some, few, wide) in ((64, limits[:4]), (128, limits[4:])):
        for row in (many, some, few, wide):
            assert row == sorted(row) and row[0] >= 16 * 4 + 64
        assert wide[0] >= 16 * 16 + 64
        assert all(a <= b <= c for a, b, c in zip(many, some, few))
    assert limits[4] == [512, 512, 576, 576] and limits[7] == [1408, 1664, 1664, 1664]
    assert limits[0] == [864, 864, 1024, 1152] and limits[3] == [3584, 5120, 5632, 7168]
