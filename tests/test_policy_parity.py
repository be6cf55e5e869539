"""Parity of the library's temporal-ROI selector (mmbev_build_rois, host
code behind the C ABI) with the oracle: ROI records bit for bit, budgets,
offsets, TTC (exact, infinity included), flags, ranks and sweep counts."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import synth
from oracle import policy as P
from test_oracle_policy import POL, as_dicts


@pytest.fixture(scope="module")
def mb():
    from paper_2608_15437_amd import mmbev

    mmbev.load()
    return mmbev


def _both(mb, d, off, e, pol):
    got = mb.build_rois(d, off, e, mb.policy(**pol))
    exp = P.build_rois(*as_dicts(d, off, e), pol)
    return got, exp


def _same(got, exp):
    assert got["roi_offsets"].tolist() == exp["roi_offsets"].tolist()
    assert np.array_equal(got["rois"].view(np.uint32).reshape(-1, 8), exp["rois"].view(np.uint32).reshape(-1, 8))
    assert np.array_equal(got["budgets"], exp["budgets"])
    assert np.array_equal(got["crit"]["ttc"], exp["ttc"])
    assert np.array_equal(got["crit"]["flags"], exp["flags"])
    assert np.array_equal(got["crit"]["rank"], exp["rank"])
    assert np.array_equal(got["sweeps"], exp["sweeps"])


@pytest.mark.parametrize("seed,frames,count,kw", [
    (1, 4, (0, 300), {}),
    (2, 8, (0, 40), {"max_optional": 5}),
    (3, 3, (100, 400), {"dense_count": 200}),
    (4, 16, (0, 12), {"dt": 0.1, "margin": 0.3, "r_coll": 3.5}),
    (5, 2, [0, 0], {}),
    (6, 2, [0, 7], {"fallback_length": 0.0}),
    (7, 5, (0, 60), {"theta_max_deg": 45.0, "theta_min_deg": 45.0, "speed_wide": 10.0, "speed_narrow": 10.0}),
])
def test_random_caches_match_oracle(mb, seed, frames, count, kw):
    d, off, e = synth.detections(seed, frames, count=count)
    _same(*_both(mb, d, off, e, dict(POL, **kw)))


def test_ties_and_exact_boundaries(mb):
    """Equal TTC and distance (order by input), objects on the cone edge and at the braking distance."""
    d = np.zeros(6, dtype=synth.DETECTION_DTYPE)
    d["length"], d["width"], d["cls"] = 4.0, 2.0, 1
    d["x"] = [10.0, 10.0, 18.75, 30.0, 30.0, 0.0]
    d["y"] = [0.0, 0.0, 0.0, 0.0, 0.0, 3.0]
    e = np.zeros(1, dtype=synth.EGO_DTYPE)
    e["speed"] = 15.0
    _same(*_both(mb, d, np.array([0, 6], np.int32), e, dict(POL)))


def _order_words(d, crit, pol):
    """Ranking keys of detections whose ego frame did not move, and the 32-bit words that order them up to ties: 30 bits
    of the TTC or, without one, of the distance."""
    x, y = d["x"] + d["vx"] * pol["dt"], d["y"] + d["vy"] * pol["dt"]
    dist, ttc, opt = np.sqrt(x * x + y * y), crit["ttc"].copy(), (crit["flags"] & 4) == 0
    bits = np.where(np.isinf(ttc), (1 << 30) | (dist.view(np.int64) >> 33), ttc.view(np.int64) >> 33)
    return list(zip(opt, ttc, dist)), bits | opt.astype(np.int64) << 31


@pytest.mark.parametrize("count,copies,theta", [(1, 1, 60.0), (64, 2, 15.0), (126, 2, 89.5), (128, 2, 90.0), (129, 3, 0.0),
                                               (128, 3, 89.0)])
def test_ranking_and_cone_edges(mb, count, copies, theta):
    """Frames up to and past the largest that is ranked by counting, with equal ranking keys (detections repeated in
    their frame) and keys that differ in their last bits only, the larger one first (one of a pair a little farther
    away), with and without a TTC; detections on the cone's edge to the last bits, and cones on both sides of the
    steepest that is decided by the tangent."""
    d, off, e = synth.detections(70 + count, 3, count=[count, 0, count])
    e["dyaw"], e["dx"], e["dy"] = 0.0, 0.0, 0.0
    d["vx"][1::4] = d["vy"][1::4] = 0.0
    d["x"][1::4] = np.abs(d["x"][1::4])
    d["y"][1::4] = d["x"][1::4] * np.tan(np.radians(theta)) * (1.0 + np.arange(len(d[1::4])) % 5 * 2.0 ** -52)
    part = count // copies
    for lo in (0, count):
        for k in range(1, copies):
            d[lo + k * part:lo + (k + 1) * part] = d[lo:lo + part]
        for k in range(lo, lo + part, 3):  # the first of the copies
            for c in ("x", "y"):
                d[c][k] += np.sign(d[c][k]) * 4 * np.spacing(abs(d[c][k]))
    pol = dict(POL, theta_max_deg=theta, theta_min_deg=theta)
    got, exp = _both(mb, d, off, e, pol)
    _same(got, exp)
    if copies > 1:  # equal words of different keys, the larger key first, with a TTC and without; equal keys
        seen = set()
        for lo in (0, count):
            key, word = _order_words(d[lo:lo + count], got["crit"][lo:lo + count], pol)
            for a in range(count):
                for b in range(a + 1, count):
                    if word[a] == word[b]:
                        seen.add((bool(np.isinf(key[a][1])), "larger" if key[a] > key[b] else "less" if key[a] < key[b] else "same"))
        assert {(True, "larger"), (True, "same"), (False, "larger"), (False, "same")} <= seen, seen


def test_rejects_bad_arguments(mb):
    d, off, e = synth.detections(9, 2, count=(3, 5))
    L = mb.load()
    for bad in ({"dt": 0.0}, {"r_coll": -1.0}, {"a_brake": 0.0}, {"theta_max_deg": 91.0},
                {"theta_min_deg": 70.0}, {"speed_wide": 40.0}, {"n_full": 256}, {"n_reduced": 11},
                {"n_reduced": 0}, {"max_optional": -1}, {"margin": float("nan")}):
        with pytest.raises(mb.MmbevError):
            mb.build_rois(d, off, e, mb.policy(**dict(POL, **bad)))
    bad_cls = d.copy()
    bad_cls["cls"][0] = 3
    bad_res = d.copy()
    bad_res["reserved"][1] = 1
    bad_nan = d.copy()
    bad_nan["vx"][2] = np.inf
    for dd in (bad_cls, bad_res, bad_nan):
        with pytest.raises(mb.MmbevError):
            mb.build_rois(dd, off, e, mb.policy(**POL))
    for oo in (np.array([1, off[1], off[2]], np.int32), np.array([0, off[2], off[1]], np.int32)):
        with pytest.raises(mb.MmbevError):
            mb.build_rois(d, oo, e, mb.policy(**POL))
    assert L.mmbev_build_rois(None, off.ctypes.data, 2, e.ctypes.data, ctypes.byref(mb.policy(**POL)), None, None,
                              None, None, None) == mb.ERR_INVALID_ARG
