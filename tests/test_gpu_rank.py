"""GPU parity of the rank walks (ensembles walked over threshold codes) with the
CPU oracle, bit for bit, at the edges of their tiles, rounds, tables and modes.
"""
import dataclasses

import numpy as np
import pytest

import gen
from paper_2411_10764_amd import ml2
from tests.test_gpu_parity import check_pipeline

pytestmark = pytest.mark.gpu

SPECIAL = np.array([np.nan, -np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-45, -1e-45, 3.4e38, -3.4e38],
                   np.float32)


def _rows(seed, n, F, K):
    """Generated rows with special values, ties and near ties sprinkled in."""
    X = gen.features(seed, n, F, K)
    rng = np.random.default_rng(seed)
    at = rng.random(X.shape)
    X = np.where(at < 0.02, rng.choice(SPECIAL, X.shape), X)
    X = np.where((at > 0.98) & (at < 0.99), np.nextafter(X, np.float32(-np.inf)), X)
    return np.ascontiguousarray(X, np.float32)


def _with_special_thresholds(ens, seed):
    rng = np.random.default_rng(seed)
    special = SPECIAL[2:]  # thresholds are never NaN
    thr = np.where(rng.random(ens.threshold.shape) < 0.03, rng.choice(special, ens.threshold.shape),
                   ens.threshold)
    return dataclasses.replace(ens, threshold=np.ascontiguousarray(thr, np.float32))


MODES = {"byte": 0, "half": 1, "packed": 2}


def _walk(ens, n, ld, perf, masked, offset=0):
    """The walk that a call takes over rows `offset` floats past an alignment."""
    e = ml2.ml2_load_ensemble(ens)
    info = ml2.ml2_probe_walk(e, 4096 + 4 * offset, n, ld, perf, masked)
    e.free()
    return info


def _assert_codes(ens, n, ld, perf, masked, mode=None, depth=0, offset=0):
    info = _walk(ens, n, ld, perf, masked, offset)
    assert info.loaded and info.codes, "the call does not walk over codes"
    assert info.depth == depth
    if mode is not None:
        assert info.mode == MODES[mode]


# Every depth in both walks: a part of a round of the chip (from 196,608 rows
# with 256 compute units a pool may rank) and one of several.
@pytest.mark.parametrize("n", [196609, 600001])
@pytest.mark.parametrize("depth,trees", [(4, 300), (5, 250), (6, 200), (7, 150), (8, 120), (9, 120),
                                         (10, 40), (11, 24), (12, 12)])
def test_every_depth(n, depth, trees):
    F, K = 40, 20
    V = _with_special_thresholds(
        gen.perfect_ensemble(15, gen.STREAM_VALIDITY, trees, depth, F, K, 0.5), 4)
    P = _with_special_thresholds(
        gen.perfect_ensemble(15, gen.STREAM_PERF, trees, depth, F, K, 0.1), 5)
    _assert_codes(V, n, F, False, False, depth=depth)
    _assert_codes(P, n, F, True, False, depth=depth)
    check_pipeline(V, P, _rows(depth, n, F, K), 16, perf_mask=False)


# a round of the chip (196,608 rows with 256 compute units) and some rows more;
# the mask of a random validity model leaves the performance walk ragged
# rounds; few features keep the pools small
@pytest.mark.parametrize("n", [196608, 196673, 270001])
@pytest.mark.parametrize("F,K,depth,trees,mode,special", [
    (24, 24, 6, 60, "byte", False),     # grids only, no table
    (33, 8, 7, 150, "packed", True),    # tables with special thresholds
    (3, 0, 10, 24, "half", False),      # tables longer than a slot
    (132, 100, 12, 3, "packed", True),  # wide rows, deepest trees, one tree per lane
])
def test_perf_walk(n, F, K, depth, trees, mode, special):
    P = gen.perfect_ensemble(11, gen.STREAM_PERF, trees, depth, F, K, 0.1)
    V = gen.perfect_ensemble(11, gen.STREAM_VALIDITY, 8, 4, F, K, 0.5)
    if special:
        P = _with_special_thresholds(P, 5)
    _assert_codes(P, n, F, True, True, mode, depth)
    check_pipeline(V, P, _rows(n, n, F, K), 16)


# fields of 4, 8 and 12 bits; of a mask, a pool of more rows ranks
@pytest.mark.parametrize("n,masked", [(196608, False), (196673, False), (450001, True)])
def test_packed_perf_walk(n, masked):
    F, K = 100, 50
    P = gen.perfect_ensemble(11, gen.STREAM_PERF, 300, 8, F, K, 0.1)
    V = gen.perfect_ensemble(11, gen.STREAM_VALIDITY, 8, 4, F, K, 0.5)
    _assert_codes(P, n, F, True, masked, "packed", 8)
    check_pipeline(V, P, _rows(n, n, F, K), 16, perf_mask=masked)


# the validity walk ranks pools of at least three quarters of a round of the
# chip (196,608 rows with 256 compute units); odd widths, strides and offsets
@pytest.mark.parametrize("n,F,K,depth,trees,ld,offset", [
    (196608, 16, 16, 4, 200, 16, 0),
    (262145, 17, 4, 5, 200, 19, 0),
    (199999, 36, 20, 6, 120, 36, 1),
    (270001, 70, 60, 8, 90, 72, 0),
    (262144, 130, 120, 9, 20, 130, 0),
])
def test_validity_walk(n, F, K, depth, trees, ld, offset):
    V = _with_special_thresholds(
        gen.perfect_ensemble(12, gen.STREAM_VALIDITY, trees, depth, F, K, 0.5), 6)
    P = gen.perfect_ensemble(12, gen.STREAM_PERF, 40, 5, F, K, 0.1)
    _assert_codes(V, n, ld, False, False, depth=depth, offset=offset)
    check_pipeline(V, P, _rows(3, n, F, K), 50, ld=ld, offset=offset)


# a plan of few float walks per lane column ranks from 64 rows per CU on
@pytest.mark.parametrize("n", [16384, 16385, 30011])
def test_deep_perf_walk_of_a_short_pool(n):
    P = _with_special_thresholds(
        gen.perfect_ensemble(14, gen.STREAM_PERF, 6, 12, 256, 128, 0.1), 5)
    V = gen.perfect_ensemble(14, gen.STREAM_VALIDITY, 8, 4, 256, 128, 0.5)
    _assert_codes(P, n, 256, True, True, "packed", 12)
    check_pipeline(V, P, _rows(n, n, 256, 128), 16)


def test_perf_walk_without_mask():
    P = gen.perfect_ensemble(13, gen.STREAM_PERF, 200, 7, 40, 20, 0.1)
    V = gen.perfect_ensemble(13, gen.STREAM_VALIDITY, 8, 4, 40, 20, 0.5)
    _assert_codes(P, 200000, 40, True, False, depth=7)
    check_pipeline(V, P, _rows(4, 200000, 40, 20), 16, perf_mask=False)


# ragged trees: byte and half-word codes, a part and more than one round (up to
# 294,912 rows), missing values with both default directions, special values
# and thresholds
@pytest.mark.parametrize("n", [294912, 400001])
@pytest.mark.parametrize("F,K,trees,depth,mode", [
    (40, 40, 90, 14, "byte"),     # grids only
    (90, 30, 120, 14, "byte"),    # tables
    (9, 0, 200, 12, "half"),
    (140, 100, 150, 20, "byte"),  # wide rows
])
def test_ragged_perf_walk(n, F, K, trees, depth, mode):
    P = gen.ragged_ensemble(21, gen.STREAM_PERF, trees, depth, F, K, 0.1, max_nodes=255)
    P = _with_special_thresholds(P, 7)
    V = gen.perfect_ensemble(21, gen.STREAM_VALIDITY, 8, 4, F, K, 0.5)
    X = _rows(n + 1, n, F, K)
    X[np.random.default_rng(8).random(X.shape) < 0.05] = np.nan
    _assert_codes(P, n, F, True, True, mode)
    check_pipeline(V, P, X, 16)


@pytest.mark.parametrize("F,K,ld,offset", [(40, 40, 40, 0), (37, 10, 41, 1)])
def test_ragged_validity_walk(F, K, ld, offset):
    n = 300003
    V = _with_special_thresholds(
        gen.ragged_ensemble(22, gen.STREAM_VALIDITY, 60, 14, F, K, 0.5, max_nodes=255), 9)
    P = gen.perfect_ensemble(22, gen.STREAM_PERF, 20, 5, F, K, 0.1)
    X = _rows(5, n, F, K)
    X[np.random.default_rng(9).random(X.shape) < 0.05] = np.nan
    _assert_codes(V, n, ld, False, False, offset=offset)
    check_pipeline(V, P, X, 50, ld=ld, offset=offset)


# ensembles and calls that the estimates leave to the float walks
@pytest.mark.parametrize("trees,depth,F,n,masked", [
    (10, 9, 132, 1000000, False),   # few deep trees over many features
    (300, 6, 128, 400000, True),    # a mask of a small pool
    (300, 6, 128, 65536, False),    # less than three quarters of a round
])
def test_float_walk_kept(trees, depth, F, n, masked):
    P = gen.perfect_ensemble(16, gen.STREAM_PERF, trees, depth, F, F // 2, 0.1)
    assert not _walk(P, n, F, True, masked).codes


def test_ragged_stumps_keep_the_float_walk():
    P = gen.ragged_ensemble(16, gen.STREAM_PERF, 20, 1, 128, 64, 0.1, max_nodes=3)
    assert not _walk(P, 1500000, 128, True, False).codes
