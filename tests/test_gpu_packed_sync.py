"""Slot tables of the packed buffer at the capacities where the synchronisation changes its launch (4096 and 8192 slots), with
updates that free and refill many slots in one call, few, or none; everything is checked by the packed-buffer test's own loop."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2605_26444_amd import synth

from test_gpu_packed import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window,nT", [(60, 4), (4000, 96), (4000, 97), (8000, 192), (8001, 192), (9000, 1200)])
def test_slots_around_the_capacity_steps(window, nT):
    V, d, M, k = 12000, 64, 3, 4
    rng = np.random.default_rng(window + nT)
    W = synth.normal_bf16(8700, 0, (V, d), 0.02)
    ctx = rng.integers(0, V, 2 * window).astype(np.int32)
    T0 = rng.choice(V, nT, replace=False).astype(np.int32)
    steps = [(rng.integers(0, V, 3), None), (np.zeros(0, np.int64), rng.choice(V, nT, replace=False)), (rng.integers(0, 50, window), None),
             (rng.choice(V, window, replace=False), rng.choice(V, nT, replace=False)), (np.full(5, 7), np.zeros(0, np.int64)), (rng.integers(0, V, 40), None)]
    _run(V, d, M, k, window, ctx, T0, steps, W, 8800)


@pytest.mark.parametrize("V,window,nT", [(20000, 16200, 184), (20000, 16200, 185), (40000, 16000, 300), (131, 100, 31), (200000, 500, 3000)])
def test_slots_beyond_them_and_at_odd_vocabulary_sizes(V, window, nT):
    """16384 slots and one more, bitmaps of five words and of more than four per thread"""
    d, M, k = 64, 3, 4
    rng = np.random.default_rng(window + nT)
    W = synth.normal_bf16(8701, 0, (V, d), 0.02)
    T = lambda: rng.choice(V, nT, replace=False).astype(np.int32)
    steps = [(rng.integers(0, V, 3), None), (np.zeros(0, np.int64), T()), (rng.choice(V, min(window, V), replace=False), T()), (rng.integers(0, V, 40), None)]
    _run(V, d, M, k, window, rng.integers(0, V, 2 * window).astype(np.int32), T(), steps, W, 8801)
