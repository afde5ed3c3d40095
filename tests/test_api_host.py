"""The host side of the library on the CPU (tests/api_host_driver.cpp): the C ABI over a
HIP runtime that can be out of device memory, with launchers that only say their name."""

import os
import shutil
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("api")
    exe, obj, plan = str(tmp / "api_host"), str(tmp / "api.o"), str(tmp / "plan.o")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-c",
                    os.path.join(ROOT, "tests", "api_host_driver.cpp"), "-o", obj], check=True)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-c", os.path.join(ROOT, "paper_2503_08461_amd", "csrc", "fc_plan.cpp"),
                    "-o", plan], check=True)
    subprocess.run(["g++", obj, plan, "-o", exe], check=True)  # (without the HIP runtime: the driver is it)
    return exe


def run(driver, scenario):
    """{what: (return code, [launches])}, and the last line as it is."""
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    lines = r.stdout.splitlines()
    out = {ln.split()[0]: (int(ln.split()[1]), ln.split()[2:]) for ln in lines if not ln.startswith("error")}
    return out, [ln for ln in lines if ln.startswith("error")]


def test_a_call_that_cannot_have_split_scores_runs_in_the_fused_kernels(driver):
    """Few long heads are split over workgroups, which takes score scratch.  Without memory for it
    the call runs as it does with many heads; the pool stays usable and no error is left behind.
    What was refused is not asked for again (an attempt waits for the device), and a captured call
    asks for nothing."""
    out, errors = run(driver, "no_room_for_split_scores")
    fused = [["plan_inline", "fused_wide+reclaim"]]
    assert out["in_place"] == (0, fused[0])
    assert out["full"] == (0, fused[0])
    assert out["full_kept_out"] == (0, fused[0])
    assert out["full_again"] == out["captured"] == (0, fused[0])
    assert errors == ["error []", "error 0", "error 0"]
    split = (0, ["plan_inline", "split_scores", "select", "gather+reclaim"])
    assert out["room"] == out["captured_warm"] == split


def test_a_pool_without_room_for_decode_segments_attends_over_whole_heads(driver):
    """A decode step over few long caches is cut into segments, whose states lie in memory of the
    pool.  A pool that cannot have it is created all the same and cuts nothing."""
    out, _ = run(driver, "no_room_for_decode_segments")
    assert out["create"][0] == 0
    assert out["whole"] == (0, ["attention_inline:1"])
    assert out["create_with_room"][0] == 0
    assert out["cut"][0] == 0 and int(out["cut"][1][0].split(":")[1]) > 1


def test_requests_of_a_decode_step(driver):
    """As arguments of the kernel where they fit, else through pinned memory, but never that in a
    captured call: a replay would read what the staging buffer holds by then."""
    out, _ = run(driver, "decode_requests")
    assert out["few"] == out["few_captured"] == (0, ["attention_inline:1"])
    assert out["many"] == (0, ["copy", "attention:1"])
    assert out["many_captured"] == (0, ["upload", "upload", "attention:1"])


def test_old_blocks_are_taken_back_exactly_once(driver):
    """By a launch of its own, or in passing by the last kernel of a call whose descriptors are
    plan_alloc's argument; only a launch is timed."""
    out, _ = run(driver, "reclaim")
    assert out["create"][0] == out["weights"][0] == 0
    main = {"fused": ["fused"], "split": ["split_scores", "select", "gather"],
            "separate": ["knorm_score", "select", "gather", "fused"], "mlp": ["mlp"]}
    before = {"few": ["plan_inline"], "many": ["upload", "upload", "plan"],
              "checked": ["upload", "zero", "check_tables", "plan"]}
    for what, kernels in main.items():
        for how, first in before.items():
            if what + "_" + how == "split_many":
                continue  # (more heads than are split)
            rc, launches = out[what + "_" + how]
            launches = [x.replace("fused_wide", "fused").replace("fused_narrow", "fused") for x in launches]
            if how == "few":
                in_passing = [k + "+reclaim" if k in ("fused", "gather", "mlp") else k for k in kernels]
                assert (rc, launches) == (0, first + in_passing)
            else:
                assert (rc, launches) == (0, first + kernels + ["reclaim"])
            assert out[what + "_" + how + "_timed"][0] == (how != "few")
