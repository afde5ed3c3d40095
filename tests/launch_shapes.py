"""Batches that run in the workgroup shape a test is about: filler requests that bring a
call's heads to the number that shape needs, and the library's own host planner
(launch_plan_driver.cpp) to say which shape every request of a call runs in."""

import functools
import os
import subprocess
import tempfile
from dataclasses import replace

import numpy as np

from conftest import ROOT
from oracle import fastcache_oracle as fo

FILLER_LEN, FILLER_BUDGET = 9, 4  # key-norm requests of nine tokens


@functools.lru_cache(None)
def _driver():
    exe = os.path.join(tempfile.mkdtemp(prefix="launch_plan"), "launch_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(ROOT, "tests", "launch_plan_driver.cpp"),
                    os.path.join(ROOT, "paper_2503_08461_amd", "csrc", "fc_plan.cpp"), "-o", exe], check=True)
    return exe


@functools.lru_cache(None)
def compute_units():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _plan(wl, methods=None, budgets=None, windows=None, lens=None, in_place=False, args=()):
    """(requests of a call that are compressed, the driver's output)"""
    methods = wl.methods if methods is None else methods
    budgets = wl.budgets if budgets is None else budgets
    windows = [wl.window] * wl.n_req if windows is None else windows
    lens = wl.seq_lens if lens is None else lens
    idx = [r for r in range(wl.n_req) if methods[r] != fo.METHOD_NONE]
    text = "%d %d %d 0 %d %d %d\n" % (wl.n_layers, wl.n_heads, wl.head_dim, in_place, compute_units(), len(idx))
    text += "".join("%d %d %d %d\n" % (lens[r], methods[r], budgets[r], windows[r]) for r in idx)
    return idx, subprocess.run([_driver(), *args], input=text, capture_output=True, text=True, check=True).stdout.splitlines()


def planned(wl, **call):
    """"split", "wide" or "narrow" for every request of a call (None: not compressed)."""
    idx, out = _plan(wl, **call)
    got = [None] * wl.n_req
    if int(out[0].split()[1]):
        for r in idx:
            got[r] = "split"
        return got
    for line in out[1::2]:
        row = [int(x) for x in line.split()[1:]]
        for i in row[5:]:
            got[idx[i]] = "wide" if row[0] else "narrow"
    return got


def pruned(wl, **call):
    """Whether a call without scores prunes each request, by the planner's lengths for its launch."""
    idx, out = _plan(wl, **call)
    methods, lens = call.get("methods", wl.methods), call.get("lens", wl.seq_lens)
    windows = call.get("windows", [wl.window] * wl.n_req)
    got = [False] * wl.n_req
    if int(out[0].split()[1]):
        return got
    for launch, limits in zip(out[1::2], out[2::2]):
        limits = [int(x) for x in limits.split()[1:]]
        for r in (idx[int(i)] for i in launch.split()[6:]):
            got[r] = methods[r] == fo.METHOD_SNAPKV and lens[r] >= limits[(windows[r] + 15) // 16 - 1]
    return got


def without_plan_alloc(wl, scores, **call):
    """Whether a call (of the default scheduling; scores: it asks for them) is one launch that reads
    the table and the stack itself."""
    return bool(int(_plan(wl, args=["one"], **call)[1][0].split()[2 if scores else 1]))


def leaves_half(wl):
    """Whether the narrow launch of a call leaves half of the keys to the caches in a pruned first pass."""
    return [bool(int(line.split()[5])) for line in _plan(wl)[1] if line.startswith("F 0")] == [True]


def in_shape(wl, shape):
    """The workload with the fillers that a call needs for `shape`: "few" none, "wide" more than
    one head per two compute units, "narrow" more than two per compute unit."""
    if shape == "few":
        return wl
    unit = wl.n_layers * wl.n_heads
    heads = compute_units() // 2 if shape == "wide" else 2 * compute_units()
    # (heads of more than 8192 tokens are in wide workgroups of their own)
    n = max(0, heads // unit + 1 - int(((wl.methods != fo.METHOD_NONE) & (wl.seq_lens <= 8192)).sum()))
    return replace(wl, seq_lens=padded(wl.seq_lens, n, FILLER_LEN), methods=padded(wl.methods, n, fo.METHOD_KNORM),
                   budgets=padded(wl.budgets, n, FILLER_BUDGET), n_blocks=wl.n_blocks + 2 * n)


def padded(a, n, value):
    return np.concatenate([np.asarray(a), np.full(n, value)]).astype(np.int32)
