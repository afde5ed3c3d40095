"""How a decode attention's heads are cut into segments (csrc/fc_plan.cpp): every
block in exactly one segment, within the room that the pool has for their states.
Host code, built with the sanitizers, no GPU."""

import os
import random
import shutil
import subprocess

import pytest

from conftest import ROOT

MAX_SEGMENTS = 16384   # of all heads of a call together
MAX_PER_HEAD = 128


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_decode_segments(tmp_path):
    exe = str(tmp_path / "decode_split")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", os.path.join(ROOT, "tests", "decode_split_driver.cpp"),
                    os.path.join(ROOT, "paper_2503_08461_amd", "csrc", "fc_plan.cpp"), "-o", exe], check=True)
    rng = random.Random(3)
    # both sides of twice the smallest segment, and nearer to two than to three of them; no tokens at all; no room
    # for two segments per head, and more than enough heads to load every compute unit alike
    cases = [(1, 4, 256, 0, [496]), (1, 4, 256, 0, [512]), (1, 4, 256, 0, [16 * 39, 5]), (1, 4, 256, 1, [0, 0]),
             (32, 257, 256, 0, [32768]),
             (32, 256, 256, 0, [32768])]
    # a CU's share of an eighth is 21 blocks, the longest head has 47: whole; 22 and 55: cut
    cases += [(1, 24, 256, 0, [16 * n] * 20 + [16 * 22] * 39) for n in (47, 55)]
    for _ in range(400):
        nl, nh = rng.choice([(1, 4), (1, 32), (2, 12), (32, 32), (80, 64)])
        cases.append((nl, nh, rng.choice([64, 256, 304]), rng.randrange(2),
                      [int(2 ** rng.uniform(0, 15)) - 1 for _ in range(rng.randrange(1, 70))]))
    text = "".join("%d %d %d %d %d %s\n" % (*c[:4], len(c[4]), " ".join(map(str, c[4]))) for c in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    got = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    assert len(got) == len(cases)
    assert [row[1] for row in got[:8]] == [1, 2, 2, 1, 1, 1, 1, 3]
    for (seg, n, *rest), (nl, nh, _, _, lens) in zip(got, cases):
        longest = (max(lens) + 15) // 16
        counts = []
        for L in lens:
            blocks, count, at = (L + 15) // 16, rest[0], rest[1:rest[0] + 2]
            rest = rest[count + 2:]
            counts.append(count)
            # one behind the other, none empty unless the head is, alike in size and near to seg
            assert at[0] == 0 and at[-1] == blocks and at == sorted(at)
            sizes = [b - a for a, b in zip(at, at[1:])]
            assert max(sizes) - min(sizes) <= 1
            if n > 1:
                assert min(sizes) > 0 or blocks == 0
                assert max(sizes) < 1.5 * seg + 1 and (count == 1 or min(sizes) >= 2 * seg // 3)
        assert not rest
        assert seg >= 1 and n == max(counts)  # no workgroups that no head has a segment for
        if n > 1:
            assert 16 <= seg <= longest // 2 and n <= MAX_PER_HEAD and n * len(lens) * nl * nh <= MAX_SEGMENTS
    assert sum(row[1] > 1 for row in got) > 50
