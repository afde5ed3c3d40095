"""The selection of a head (csrc/fc_unit.h: select_unit, bound_classify) run lane by
lane on the CPU, wavefronts and lanes in every extreme order, against a plain
statement of what it selects: the code as it is compiled for the GPU, no GPU."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")

ALL_KEYS = (0, 0xFFFFFFFF)
ORDERS = range(4)  # bit 0: lanes, bit 1: wavefronts from the highest down


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("select") / "select_emulation")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1",
                    os.path.join(ROOT, "tests", "select_emulation_driver.cpp"), "-o", exe], check=True)
    return exe


def score_keys(scores):
    """uint32 in the order of the floats, -0 and +0 alike."""
    u = (np.asarray(scores, np.float32) + np.float32(0)).view(np.uint32)
    return np.where(u >> 31, ~u, u | 0x80000000)


def pooled(scores, width):
    """Max-pooled, what is not a number left out of a maximum with numbers."""
    h = width // 2
    p = np.pad(scores, h, mode="edge")  # (a window over an end holds the token there)
    return np.fmax.reduce([p[i:i + len(scores)] for i in range(width)])


def kept_tokens(scores, k):
    """The k best scores, ties to the lower index, in token order."""
    order = np.argsort(-score_keys(scores).astype(np.int64), kind="stable")
    return np.sort(order[:k])


class Case:
    def __init__(self, scores, k, width=7, snap=True, window=3, waves=4, hints=ALL_KEYS, order=0, bounds=None):
        self.scores = np.asarray(scores, np.float32)
        self.k, self.width, self.snap, self.window = k, width, snap, window if snap else 0
        self.waves, self.hints, self.order, self.bounds = waves, hints, order, bounds

    def text(self):
        n = len(self.scores)
        head = "%d %d %d %d %d %d %x %x %d %d" % (self.waves, self.snap, n, self.window, self.k, self.width,
                                                  self.hints[0], self.hints[1], self.bounds is not None, self.order)
        words = [] if self.bounds is None else [self.bounds]
        return "\n".join([head] + [" ".join("%x" % w for w in x) for x in [self.scores.view(np.uint32)] + words])

    def __repr__(self):
        return "n %d k %d width %d snap %d waves %d order %d" % (len(self.scores), self.k, self.width, self.snap,
                                                                 self.waves, self.order)


def run(driver, cases):
    """[(key_lo, key_hi, kept, scores, named)] of the cases."""
    r = subprocess.run([driver], input="\n".join(c.text() for c in cases), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, "%s (after %d cases)" % (r.stdout[-200:], r.stdout.count("\n") // 4)
    lines = r.stdout.split("\n")
    out = []
    for i in range(len(cases)):
        keys, kept, scores, named = (lines[4 * i + j].split() for j in range(4))
        out.append((int(keys[0], 16), int(keys[1], 16), np.array(kept, np.int64),
                    np.array([int(x, 16) for x in scores], np.uint32).view(np.float32), np.array(named, np.int64)))
    return out


def check(driver, cases):
    for c, (_, _, kept, scores, _) in zip(cases, run(driver, cases)):
        n = len(c.scores)
        final = pooled(c.scores, c.width) if c.snap else c.scores
        np.testing.assert_array_equal(scores[:n], final, str(c))
        assert (scores[n:] == np.inf).all(), c
        want = np.concatenate([kept_tokens(final, c.k), n + np.arange(c.window)])
        np.testing.assert_array_equal(kept, want, str(c))


@pytest.mark.parametrize("waves", [4, 12, 16])
def test_selection(driver, waves):
    """Counts at the edges of a lane's four tokens, of a chunk and of a segment, every kind of
    pooling width, values that tie, one candidate list and many."""
    rng = np.random.default_rng(waves)
    cases = []
    for i, n in enumerate([1, 2, 5, 63, 255, 256, 257, 1023, 1025, 64 * waves * 4 + 3, 2048, 2049, 3600]):
        for width in (1, 3, 7, 9, 17, 63):
            kinds = [rng.random(n), rng.integers(0, 9, n) / 8.0, 1.0 + rng.random(n) * 1e-5,
                     2.0 ** rng.integers(-60, 3, n)]
            cases.append(Case(kinds[(i + width) % 4], int(rng.integers(0, n + 1)), width, waves=waves,
                              order=int(rng.integers(0, 4))))
        cases.append(Case(-rng.random(n), max(1, n // 2), snap=False, waves=waves, order=i % 4))
    check(driver, cases)


@pytest.mark.parametrize("order", ORDERS)
def test_a_range_that_is_a_single_key(driver, order):
    """The hinted range narrowed to one key that few tokens have: neither histogram nor candidate
    list, nothing to wait for between the counts of one step and of the next."""
    rng = np.random.default_rng(5)
    for waves in (4, 16):
        scores = np.ones(1500, np.float32)
        places = rng.permutation(1500)
        scores[places[:60]] = 3.0
        scores[places[60:100]] = 2.0
        key = int(score_keys([2.0])[0])
        check(driver, [Case(scores, 80, 1, waves=waves, hints=(key, key), order=order)])


def test_scores_that_are_not_numbers_still_fill_the_budget(driver):
    """Scores with every bit set, as a buffer of log-sum-exps that was never written gives: the
    lowest of all, the lowest indices first, and no key that stands for "no token"."""
    ones = np.full(1, 0xFFFFFFFF, np.uint32).view(np.float32)[0]
    cases = []
    for snap in (True, False):
        for n, k in ((40, 10), (700, 300), (2049, 2000)):
            scores = np.full(n, ones, np.float32)
            cases.append(Case(scores, k, 1, snap=snap))
            scores = scores.copy()
            scores[::5] = -np.arange(len(scores[::5])) if not snap else np.arange(len(scores[::5]))
            cases.append(Case(scores, k, 1, snap=snap, order=1))
    check(driver, cases)


@pytest.mark.parametrize("bits", [0x7FC00000, 0xFFC00000])
def test_pooling_leaves_out_what_is_not_a_number(driver, bits):
    """With the log-sum-exps handed in, a key row that is not a number spoils its own token's sum
    only: the windows around it hold the largest of the others."""
    nan = np.full(1, bits, np.uint32).view(np.float32)[0]
    rng = np.random.default_rng(bits & 7)
    cases = []
    for n in (5, 64, 700, 2049):
        for width in (1, 3, 5, 7, 9, 17, 63):
            scores = rng.random(n).astype(np.float32)
            scores[rng.random(n) < (0.1, 0.6)[width % 4 == 1]] = nan
            if n == 700:
                scores[:90] = scores[-90:] = nan     # whole windows, the ends among them
            cases.append(Case(scores, max(1, n // 3), width, order=width % 4))
    check(driver, cases)


@pytest.mark.parametrize("within", [1, 63, 64, 65, 255, 256, 257, 900])
def test_hinted_ranges(driver, within):
    """A range known to hold the threshold, with as many keys as are listed at once, ranked at
    once, and more; the threshold at either end of it and in the middle."""
    rng = np.random.default_rng(within)
    cases = []
    for waves in (4, 16):
        n, above = 1500, 200
        for place, k in enumerate((above + 1, above + (within + 1) // 2, above + within)):
            scores = np.empty(n, np.float32)
            at = rng.permutation(n)
            scores[at[:above]] = 4.0 + rng.random(above)
            scores[at[above:above + within]] = 2.0 + rng.random(within)
            scores[at[above + within:]] = rng.random(n - above - within)
            cases.append(Case(scores, k, 1, waves=waves, order=place,
                              hints=tuple(int(x) for x in score_keys([2.0, 3.0]))))
            # (and with hints that turn out not to hold it: nothing is narrowed)
            cases.append(Case(scores, above, 1, waves=waves, order=place,
                              hints=tuple(int(x) for x in score_keys([2.0, 3.0]))))
    check(driver, cases)


def packed(lo, hi):
    """Upper bounds rounded up, lower bounds down to their leading 16 bits, one word each."""
    up = (np.asarray(hi, np.float32).view(np.uint32).astype(np.uint64) + 0xFFFF) >> 16
    return (up << 16 | np.asarray(lo, np.float32).view(np.uint32) >> 16).astype(np.uint32)


@pytest.mark.parametrize("waves", [4, 12, 16])
@pytest.mark.parametrize("width", [1, 7, 9, 63])
def test_selection_through_bounds(driver, waves, width):
    """Bounds that are tight, loose, skewed or trivial, values that tie or span 2^60: with the named
    tokens re-scored and upper bounds elsewhere, what is kept is what exact scores would keep, the
    hinted keys enclose the threshold, and a token decided by its own bounds is not named."""
    rng = np.random.default_rng(100 * waves + width)
    cases, share = [], []
    for i, n in enumerate([3, 40, 255, 256, 257, 600, 1025, 2049, 3600] * 3):
        kinds = [np.exp(rng.normal(0, 1.5, n)), rng.integers(1, 9, n) / 8.0, 1.0 + rng.random(n) * 1e-5,
                 2.0 ** rng.integers(-60, 3, n), np.ones(n), np.where(rng.random(n) < 0.01, 3.0, 1e-20 * rng.random(n))]
        x = kinds[i % 6].astype(np.float32)
        slack, skew = rng.random(n) * (0.0, 0.01, 0.3, 1.0)[i % 4], (0.05, 0.5, 0.95)[i % 3]
        trivial = rng.random(n) < (0.0, 0.05, 0.0, 1.0)[(i + 1) % 4]
        lo = np.minimum(np.where(trivial, 0.0, x * (1.0 - slack * skew)).astype(np.float32), x)
        hi = np.maximum(np.where(trivial, 64.0, x * (1.0 + 3.0 * slack * (1.0 - skew))).astype(np.float32), x)
        cases.append(Case(x, int(rng.integers(1, n)), width, waves=waves, order=i % 4, bounds=packed(lo, hi)))
    for c, (key_lo, key_hi, kept, _, named) in zip(cases, run(driver, cases)):
        final = pooled(c.scores, c.width)
        np.testing.assert_array_equal(kept, np.concatenate([kept_tokens(final, c.k), len(final) + np.arange(c.window)]), str(c))
        threshold = np.sort(score_keys(final))[-c.k]
        assert key_lo <= threshold <= key_hi, c
        up, low = score_keys((c.bounds & 0xFFFF0000).view(np.float32)), score_keys((c.bounds << 16).view(np.float32))
        np.testing.assert_array_equal(named, (up >= key_lo) & (low <= key_hi), str(c))
        share.append(named.mean())
    assert min(share) < 0.1 and max(share) == 1.0
