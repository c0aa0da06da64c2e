"""GPU parity of the rank walks (ensembles walked over threshold codes) with the
CPU oracle, bit for bit, at the edges of their tiles, rounds, tables and modes.
"""
import dataclasses

import numpy as np
import pytest

import gen
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


# a round of the chip (196,608 rows with 256 compute units take the rank walk)
# and some rows more; the mask of a random validity model leaves the
# performance walk ragged rounds; few features keep the pools small
@pytest.mark.parametrize("n", [196608, 196673, 270001])
@pytest.mark.parametrize("F,K,depth,trees,special", [
    (24, 24, 6, 60, False),   # byte tile, grids only, no table
    (33, 8, 7, 150, True),    # byte tile or packed: tables with special thresholds
    (100, 50, 8, 300, False), # packed tile: 4-, 8- and 12-bit fields
    (3, 0, 10, 24, False),    # half-word tile: tables longer than a slot
    (132, 100, 12, 3, True),  # wide rows, deepest trees, one tree per lane
])
def test_perf_walk(n, F, K, depth, trees, special):
    P = gen.perfect_ensemble(11, gen.STREAM_PERF, trees, depth, F, K, 0.1)
    V = gen.perfect_ensemble(11, gen.STREAM_VALIDITY, 8, 4, F, K, 0.5)
    if special:
        P = _with_special_thresholds(P, 5)
    check_pipeline(V, P, _rows(n, n, F, K), 16)


# the validity walk ranks pools of at least three quarters of a round of the
# chip (196,608 rows with 256 compute units); odd widths, strides and offsets
@pytest.mark.parametrize("n,F,K,depth,trees,ld,offset", [
    (196608, 16, 16, 4, 20, 16, 0),
    (262145, 17, 4, 5, 90, 19, 0),
    (199999, 36, 20, 6, 120, 36, 1),
    (270001, 70, 60, 8, 90, 72, 0),
    (262144, 130, 120, 9, 20, 130, 0),
])
def test_validity_walk(n, F, K, depth, trees, ld, offset):
    V = _with_special_thresholds(
        gen.perfect_ensemble(12, gen.STREAM_VALIDITY, trees, depth, F, K, 0.5), 6)
    P = gen.perfect_ensemble(12, gen.STREAM_PERF, 40, 5, F, K, 0.1)
    check_pipeline(V, P, _rows(3, n, F, K), 50, ld=ld, offset=offset)


# a plan of few float walks per lane column ranks from 64 rows per CU on
@pytest.mark.parametrize("n", [16384, 16385, 30011])
def test_deep_perf_walk_of_a_short_pool(n):
    P = gen.perfect_ensemble(14, gen.STREAM_PERF, 6, 12, 256, 128, 0.1)
    V = gen.perfect_ensemble(14, gen.STREAM_VALIDITY, 8, 4, 256, 128, 0.5)
    check_pipeline(V, _with_special_thresholds(P, 5), _rows(n, n, 256, 128), 16)


def test_perf_walk_without_mask():
    P = gen.perfect_ensemble(13, gen.STREAM_PERF, 200, 7, 40, 20, 0.1)
    V = gen.perfect_ensemble(13, gen.STREAM_VALIDITY, 8, 4, 40, 20, 0.5)
    check_pipeline(V, P, _rows(4, 200000, 40, 20), 16, perf_mask=False)


# ragged trees: byte and half-word codes, a part and more than one round (up to
# 294,912 rows), missing values with both default directions, special values
# and thresholds
@pytest.mark.parametrize("n", [294912, 400001])
@pytest.mark.parametrize("F,K,trees,depth", [
    (40, 40, 90, 14),    # byte codes, grids only
    (90, 30, 120, 14),   # byte codes, tables
    (9, 0, 200, 12),     # half-word codes
    (140, 100, 50, 20),  # wide rows
])
def test_ragged_perf_walk(n, F, K, trees, depth):
    P = gen.ragged_ensemble(21, gen.STREAM_PERF, trees, depth, F, K, 0.1, max_nodes=255)
    P = _with_special_thresholds(P, 7)
    V = gen.perfect_ensemble(21, gen.STREAM_VALIDITY, 8, 4, F, K, 0.5)
    X = _rows(n + 1, n, F, K)
    X[np.random.default_rng(8).random(X.shape) < 0.05] = np.nan
    check_pipeline(V, P, X, 16)


@pytest.mark.parametrize("F,K,ld,offset", [(40, 40, 40, 0), (37, 10, 41, 1)])
def test_ragged_validity_walk(F, K, ld, offset):
    n = 300003
    V = _with_special_thresholds(
        gen.ragged_ensemble(22, gen.STREAM_VALIDITY, 60, 14, F, K, 0.5, max_nodes=255), 9)
    P = gen.perfect_ensemble(22, gen.STREAM_PERF, 20, 5, F, K, 0.1)
    X = _rows(5, n, F, K)
    X[np.random.default_rng(9).random(X.shape) < 0.05] = np.nan
    check_pipeline(V, P, X, 50, ld=ld, offset=offset)
