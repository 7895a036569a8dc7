"""The bootstrap's replicates together at the sizes of their workspace: target temperatures in
several passes, replicates in several batches, the most values of N that a block holds."""
import numpy as np
import pytest

import oracle
from paper_1908_11118_amd import regc
from paper_1908_11118_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    torch.cuda.set_device(0)


def _records(t, mu, n_max, centre, recs, seed):
    """Whole records of a gas with Poisson N (mean `centre` at the middle state) and energies
    around -0.02 N."""
    rng = np.random.default_rng(seed)
    lnz = np.array([[m / x + 1.5 * np.log(x) for m in mu] for x in t]).ravel()
    n = np.minimum(rng.poisson(centre * np.exp(lnz - np.median(lnz)), (recs, len(lnz))), n_max).astype(np.int32)
    e = -0.02 * n + rng.normal(0.0, 0.3, n.shape)
    s = np.broadcast_to(np.arange(len(lnz), dtype=np.int32), n.shape)
    return e.ravel(), n.ravel(), s.ravel().copy()


def test_target_temperatures_in_several_passes():
    """4000 target temperatures at once would need 2.8 GB for 128 replicates: the workspace
    stays below its bound, is not kept, and every target's error is that of a call for a few."""
    import torch
    t, mu = W.linear_grid(1.2, 1.4, 3), W.linear_grid(-3.2, -3.0, 3)
    e, n, s = _records(t, mu, 24, 9.0, 40, 1)
    tt, tm = W.linear_grid(1.2, 1.4, 4000), np.array([-3.15, -3.05])
    mb = regc.Mbar(t, mu, 24)
    mb.set_samples(e, n, s)
    mb.reweight(tt[:2], tm, tol=1e-12, n_boot=128)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    got = mb.reweight(tt, tm, tol=1e-12, n_boot=128)
    torch.cuda.synchronize()
    kept = free - torch.cuda.mem_get_info()[0]
    for a in (0, 1500, 3990):
        part = mb.reweight(tt[a: a + 10], tm, tol=1e-12, n_boot=128)
        for name in ("se_n", "se_heat_cap"):
            assert np.array_equal(got[name].reshape(4000, 2)[a: a + 10], part[name].reshape(10, 2)), (a, name)
    mb.close()
    assert kept < 64 << 20


# 128 replicates make a batch; 512 and 1024 values of N take 64 and 128 KB in a block, 1025 go
# one replicate after the other
@pytest.mark.parametrize("n_boot,n_max,centre", [(128, 40, 20.0), (129, 40, 20.0), (145, 40, 20.0), (20, 511, 300.0),
                                                 (20, 512, 300.0), (20, 1023, 700.0), (17, 1024, 700.0)])
def test_batches_and_values_of_n(n_boot, n_max, centre):
    t, mu = W.linear_grid(1.28, 1.32, 2), W.linear_grid(-3.12, -3.08, 3)
    recs = 30
    e, n, s = _records(t, mu, n_max, centre, recs, n_boot)
    w = W.ideal_gas().replace(t=t, mu=mu, n_max=n_max)
    tt, tm = [1.29, 1.31], [-3.11, -3.09]
    mb = regc.Mbar(t, mu, n_max)
    mb.set_samples(e, n, s)
    got = mb.reweight(tt, tm, tol=1e-12, n_boot=n_boot, seed=5, n_sites=8.0)
    mb.close()
    beta, lnz = oracle.state_arrays(w)
    f, _, ok, _, _ = oracle.mbar_solve(beta, lnz, np.bincount(s, minlength=6), e, n, tol=1e-12, max_iter=100000)
    tb, tz = np.repeat(1.0 / np.array(tt), 2), np.array([oracle.state_lnz(a, b) for a in tt for b in tm])
    se_n, se_c, _, _, conv = oracle.mbar_bootstrap(beta, lnz, e, n, s, 6, max(1, recs // 20), n_boot, 5, f, tb, tz, n_max,
                                                  tol=1e-12)
    assert ok and conv and got["converged"]
    assert np.allclose(got["se_n"], se_n, rtol=1e-5, atol=0)
    assert np.allclose(got["se_heat_cap"], se_c, rtol=1e-4, atol=0)


@pytest.mark.parametrize("record_size,block,recs", [(1, 1, 20), (1, 7, 20), (2, 1, 30), (6, 30, 30), (6, 29, 30), (1, 0, 300)])
def test_records_and_blocks(record_size, block, recs):
    """Blocks of one record, of all records, and with a remainder."""
    t, mu = W.linear_grid(1.28, 1.32, 2), W.linear_grid(-3.12, -3.08, 3)
    e, n, s = _records(t, mu, 30, 12.0, recs, block)
    w = W.ideal_gas().replace(t=t, mu=mu, n_max=30)
    tt, tm = [1.3], [-3.11, -3.09]
    mb = regc.Mbar(t, mu, 30)
    mb.set_samples(e, n, s)
    got = mb.reweight(tt, tm, tol=1e-12, n_boot=9, record_size=record_size, block_records=block, seed=11)
    mb.close()
    beta, lnz = oracle.state_arrays(w)
    f, _, ok, _, _ = oracle.mbar_solve(beta, lnz, np.bincount(s, minlength=6), e, n, tol=1e-12, max_iter=100000)
    tb, tz = np.repeat(1.0 / np.array(tt), 2), np.array([oracle.state_lnz(tt[0], b) for b in tm])
    R = len(e) // record_size
    se_n, se_c, _, _, conv = oracle.mbar_bootstrap(beta, lnz, e, n, s, record_size, block or max(1, R // 20), 9, 11, f, tb, tz,
                                                  30, tol=1e-12)
    assert ok and conv and got["converged"]
    assert np.allclose(got["se_n"], se_n, rtol=1e-5, atol=1e-12)
    assert np.allclose(got["se_heat_cap"], se_c, rtol=1e-4, atol=1e-12)


def test_many_blocks_take_no_longer_than_few():
    """2e6 records: the blocks' draws, one by one, took a second for blocks of one record and
    20 ms for blocks of 10 000."""
    import time
    t, mu = W.linear_grid(1.2, 1.4, 8), W.linear_grid(-3.2, -3.0, 8)
    e, n, s = _records(t, mu, 24, 9.0, 31250, 2)
    mb = regc.Mbar(t, mu, 24)
    mb.set_samples(e, n, s)
    took = {}
    for block in (10000, 1):
        runs = []
        for _ in range(3):
            t0 = time.perf_counter()
            mb.reweight([1.25, 1.3], [-3.1], tol=1e-10, n_boot=100, record_size=1, block_records=block)
            runs.append(time.perf_counter() - t0)
        took[block] = min(runs)
    mb.close()
    assert took[1] < 5 * took[10000] + 0.05
