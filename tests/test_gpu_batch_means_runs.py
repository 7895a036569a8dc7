"""Batch means of samples that come sorted by state, whole or in part: waves that see one
state (of one batch, of several), waves whose share begins so and goes on otherwise."""
import time

import numpy as np
import pytest

import oracle
from paper_1908_11118_amd import regc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    torch.cuda.set_device(0)


@pytest.mark.parametrize("n_states,n_samples,n_batches", [(1, 70000, 7), (1, 300000, 3000), (5, 200001, 20), (64, 500000, 20),
                                                          (700, 300000, 20), (1366, 300000, 9), (2731, 300000, 9)])
@pytest.mark.parametrize("mixed", [0.0, 0.3])
def test_samples_sorted_by_state(n_states, n_samples, n_batches, mixed):
    rng = np.random.default_rng(n_samples + n_states)
    state = np.sort(rng.integers(0, n_states, n_samples)).astype(np.int32)
    # every third stretch of 1000 samples is in any order
    any_order = (np.arange(n_samples) // 1000 % 3 == 2) & (mixed > 0)
    state[any_order] = rng.integers(0, n_states, any_order.sum())
    n = rng.integers(0, 500, n_samples).astype(np.int32)
    n[::7] = 2 ** 31 - 1
    mean, se = regc.batch_means(state, n, n_states, n_batches)
    ref_mean, ref_se = oracle.batch_means(n_states, state, n, n_batches)
    assert np.array_equal(np.isnan(mean), np.isnan(ref_mean))
    assert np.allclose(mean, ref_mean, rtol=1e-13, atol=0, equal_nan=True)
    assert np.allclose(se, ref_se, rtol=1e-10, atol=1e-13 * 2.0 ** 31, equal_nan=True)


def test_sorted_samples_take_no_longer_than_the_sort():
    """4e6 samples of 64 states: 120 us in any order, 710 us in the order of the states."""
    import torch
    state = np.random.default_rng(0).integers(0, 64, 4000000).astype(np.int32)
    took = []
    for order in (state, np.sort(state)):
        s, n = torch.from_numpy(order).cuda(), torch.from_numpy(state).cuda()
        runs = []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            regc.batch_means(s, n, 64, 20)
            runs.append(time.perf_counter() - t0)
        took.append(min(runs))
    assert took[1] < 2.5 * took[0]
