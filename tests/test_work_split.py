"""The kernel's rule for cutting a call's work (csrc/rlda_split.h), compiled for the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2607_09207_amd as pkg
from paper_2607_09207_amd import calibrate as C

CSRC = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "csrc")
FORMS = {"full": 0, "half128": 1, "half64": 2, "general": 3}
START = 2   # pages a segment's start costs


class Split(ctypes.Structure):
    _fields_ = [("whole", ctypes.c_bool), ("shares", ctypes.c_int)]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "rule.cpp").write_text('''#include "rlda_split.h"
extern "C" rlda::Split split(int form, int W, int nseg, int cost, int nb) {
  return rlda::split_of((rlda::SplitForm)form, W, 1.f / W, nseg, cost, nb);
}
extern "C" rlda::Split forced(int W, int nseg, int cost, int nb) {
  return rlda::split_of(rlda::kSplitFullPages, W, 0.f, nseg, cost, nb);
}
extern "C" int share(int b, int n) { return rlda::share_of_block(b, n); }
''')
    so = str(d / "rule.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "rule.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    lib.split.restype = lib.forced.restype = Split
    return lib


def equal(rule, form, W, nseg, nb):
    """The cut of nseg segments of nb pages."""
    return rule.split(FORMS[form], W, nseg, nseg * (nb + START), nb)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 18, 29, 38, 116, 255, 256])
def test_the_shares_in_use_are_spread_over_the_xcds(rule, n):
    shares = [rule.share(b, n) for b in range(256)]
    assert sorted(s for s in shares if s >= 0) == list(range(n))
    per_xcd = [[s for s in shares[x::8] if s >= 0] for x in range(8)]
    assert max(map(len, per_xcd)) - min(map(len, per_xcd)) <= 1
    assert all(s == list(range(s[0], s[0] + len(s))) for s in per_xcd if s)   # neighbours on one XCD


def test_a_forced_share_count_is_kept(rule):
    s = rule.forced(7, 4, 40, 8)
    assert not s.whole and s.shares == 7


@pytest.mark.parametrize("nb", [1, 8, 62, 63, 64, 112, 188, 300, 310, 1000, 2048])
@pytest.mark.parametrize("nseg", [1, 2, 3, 8, 13])
def test_few_segments_fall_into_one_merge_batch(rule, nseg, nb):
    """Alone, a segment is cut into at most 16 pieces, shares of at least 4 pages; above
    300 pages into at most (nb + START) / sqrt(1.25 nb); a multiple of the segments."""
    s = equal(rule, "full", 256, nseg, nb)
    pieces = s.shares / nseg
    if s.shares < 256:
        assert pieces == int(pieces) >= 1
        assert pieces <= max(16, -(-(nb + START) // (1.25 * nb) ** 0.5))
        assert pieces == 1 or (nb + START) / (pieces - 1) >= 4


@pytest.mark.parametrize("form", ["full", "half128", "general"])
def test_unlike_segments_keep_the_workgroups_unless_clearly_fewer_do(rule, form):
    W = 256
    for nseg in (4, 12, 41):
        for nb in (200, 344, 726):
            for mean in range(20, nb, 7):
                cost = nseg * (mean + START)
                s = rule.split(FORMS[form], W, nseg, cost, nb)
                assert s.shares == W or s.shares <= 0.7 * W, (nseg, nb, mean)
    # 164 segments of up to 344 pages, 12 of up to 726: 492 of 512 and 216 of 256 shares by the bound on their pages
    assert rule.split(FORMS["half128"], 512, 164, 9408, 344).shares == 512
    assert rule.split(FORMS["full"], 256, 12, 6180, 726).shares == 256
    assert equal(rule, "full", 256, 12, 500).shares == 252   # of one length: cut alike


@pytest.mark.parametrize("nb", [1, 64, 112])
def test_shares_that_are_the_segments_stay_shares_in_the_general_loop(rule, nb):
    """As many segments as workgroups, all of one length: cut nothing, gain nothing."""
    s = equal(rule, "general", 256, 256, nb)
    assert not s.whole and s.shares == 256
    assert rule.split(FORMS["general"], 256, 256, 256 * (nb + START) - 1, nb).whole   # one page less in one of them
    assert equal(rule, "general", 256, 255, nb).whole
    assert equal(rule, "full", 256, 256, nb).whole


# (form, segments of 256 workgroups, pages over an equal share that still go whole)
LINES = [("full", 4, 52.875), ("full", 128, 26), ("full", 256, 26), ("half128", 32, 57), ("half128", 128, 77),
         ("half64", 32, 78), ("half64", 256, 138), ("general", 16, 40), ("general", 64, 22), ("general", 255, 20)]


@pytest.mark.parametrize("form,nseg,over", LINES)
def test_both_sides_of_each_line(rule, form, nseg, over):
    W = 256
    whole = [nb for nb in range(1, 2000) if rule.split(FORMS[form], W, nseg, 256 * 40, nb).whole]
    assert whole == list(range(1, 1 + int(over + 40)))   # the equal share is 40 pages
    assert not rule.split(FORMS[form], W, W + 1, (W + 1) * 3, 1).whole


@pytest.mark.parametrize("form,kv,d", [("full", "bf16", 128), ("half128", "fp8_e4m3fn", 128), ("half64", "bf16", 64),
                                       ("half64", "fp8_e4m3fn", 64), ("full", "f32", 64)])
def test_the_predictor_mirrors_the_rule(rule, form, kv, d):
    rng = np.random.default_rng(5)
    differ = 0
    for _ in range(3000):
        hkv, W = int(rng.integers(1, 9)), int(rng.choice([64, 256, 512]))
        lens = np.exp(rng.uniform(0, np.log(20000), int(rng.integers(1, 80)))).astype(int) * (rng.random() < 0.98)
        n = (lens + 15) // 16
        cost = hkv * int(n.sum() + START * np.count_nonzero(n))
        got = rule.split(FORMS[form], W, len(lens) * hkv, cost, int(n.max()))
        whole, shares = C.work_split(lens, hkv, W, d, kv)
        differ += (got.whole, got.shares) != (whole, shares)
    assert differ <= 3   # fp32 against float64, within rounding of a line


def test_a_small_table_bounds_the_workgroups():
    """One page a sequence: no more workgroups than pages, as the host launches."""
    assert C.work_split([5] * 3, 2, 256, 128, "bf16", max_pages=1) == C.work_split([5] * 3, 2, 6, 128, "bf16")
    assert C.work_split([500], 1, 256, 128, "bf16", max_pages=32) == C.work_split([500], 1, 32, 128, "bf16")
    assert C.work_split([500], 1, 256, 128, "bf16", max_pages=1000) == C.work_split([500], 1, 256, 128, "bf16")


def test_pieces_of_the_chosen_cut():
    assert C.features_ext([500] * 4, 4, 256, 128, "bf16")[3] == 1           # whole segments
    assert C.features_ext([3000], 1, 256, 128, "bf16")[3] == 16             # one segment alone
    assert C.features_ext([3000], 1, 256)[3] == C.max_pieces([3000], 1, 256) > 100   # 256 shares
