"""What regc_mbar_solve promises: converged means max |delta f| < tol, whatever iteration the
limit falls on and however the residual moves about near its rounding."""
import numpy as np
import pytest

import oracle
from paper_1908_11118_amd import regc
from paper_1908_11118_amd import workloads as W
from test_gpu_mbar_solve import fluid_samples

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    torch.cuda.set_device(0)


def _loaded(t, mu, n_max, per_state, seed, spread=1.0):
    e, n, s = fluid_samples(t, mu, n_max, per_state, seed=seed, spread=spread)
    mb = regc.Mbar(t, mu, n_max)
    mb.set_samples(e, n, s)
    return mb, e, n, s


# grids of more than 32 temperatures and limits below 64 take the plain iteration, the others
# the preconditioned one; the residual rises past tol again in the first and last three
# (tolerances near its rounding, and loose ones)
@pytest.mark.parametrize("n_t,n_mu,n_max,per_state,spread,cold,seed,tols,limits", [
    (3, 5, 77, 52, 2.0, False, 11, (3.15e-14, 4.97e-14, 7.84e-14), (63, 400)),
    (33, 3, 50, 50, 1.0, True, 0, (2e-14, 1e-10, 1e-4), range(100, 160, 3)),
    (6, 6, 38, 36, 0.5, False, 1, (1e-12, 1e-7, 1e-2), range(1, 80, 4)),
    (40, 4, 65, 66, 0.5, True, 82, (1e-1,), range(44, 58)),
    (40, 4, 82, 32, 1.0, True, 18, (3.15e-14, 7.84e-14), (400,)),
    (3, 5, 87, 30, 1.0, False, 411, (1e-1, 1e-2, 1e-5), (400,))])
def test_converged_means_below_the_tolerance(n_t, n_mu, n_max, per_state, spread, cold, seed, tols, limits):
    t = W.linear_grid(0.6, 1.4, n_t) if cold else W.linear_grid(0.8, 1.8, n_t)
    mu = W.linear_grid(-6.0, -2.0, n_mu) if cold else W.linear_grid(-5.0, -2.5, n_mu)
    mb, e, n, s = _loaded(t, mu, n_max, per_state, seed, spread)
    beta, lnz = oracle.state_arrays(W.ideal_gas().replace(t=t, mu=mu, n_max=n_max))
    omega = np.bincount(s, minlength=len(beta))
    seen = 0
    for tol in tols:
        for limit in limits:
            f, conv, it, d = mb.solve(tol=tol, max_iter=limit, allow_noconv=True)
            if conv:
                seen += 1
                assert d < tol, (tol, limit, it, d)
                # (f is a map value; a further step of the map moves it no farther than a few
                # times the step before, to the rounding of f)
                g, _ = oracle.mbar_iterate(beta, lnz, omega, e, n, f)
                assert np.max(np.abs(g - g[0] - f)) < 10 * d + 1e-11, (tol, limit, it, d)
    mb.close()
    assert seen


# (sampled so that the first phase of the preconditioned solve takes long; in the last case it
# is given up)
@pytest.mark.parametrize("n_t,n_mu,n_max,per_state,spread,cold,seed", [
    (10, 3, 151, 67, 1.0994678737814576, 0.7119762452586738, 15), (2, 18, 98, 60, 0.7877822813860588, 0.5167166455213299, 67),
    (10, 5, 158, 98, 1.352980275804317, 0.5605383714956059, 259), (11, 4, 143, 143, 0.9377045405814164, 0.5293343299291084, 568),
    (4, 4, 92, 100, 1.0, 0.6, 4)])
def test_iterations_stay_within_the_limit(n_t, n_mu, n_max, per_state, spread, cold, seed):
    t, mu = W.linear_grid(cold, 1.6, n_t), W.linear_grid(-6.0, -2.0, n_mu)
    mb, *_ = _loaded(t, mu, n_max, per_state, seed, spread)
    for tol in (1e-6, 1e-13):
        for limit in (64, 65, 70, 90, 119, 1000):
            f, conv, it, d = mb.solve(tol=tol, max_iter=limit, allow_noconv=True)
            ms, counted = mb.timing()
            assert it <= limit and counted >= it
            assert conv == (d < tol) and (conv or it == limit)
    mb.close()


def test_a_limit_reached_on_wide_energies_is_not_run_twice():
    """Exponents between 300 and 350, where a sum may overflow: a solve that ends at the limit
    without a map value that is not finite is final (its time is that of the same samples with
    narrow energies; the general iteration after it took as long again and more)."""
    import time
    t, mu = W.linear_grid(0.05, 2.0, 32), W.linear_grid(-2.6, -2.4, 32)
    rng = np.random.default_rng(9)
    ns = 400000
    n = rng.integers(0, 6, ns).astype(np.int32)
    s = rng.integers(0, 1024, ns).astype(np.int32)
    took = {}
    for shift in (20.0, 58.0):
        e = rng.normal(0.0, 1.0, ns)
        e[:40] += shift
        mb = regc.Mbar(t, mu, 5)
        mb.set_samples(e, n, s)
        runs = []
        for _ in range(4):
            t0 = time.perf_counter()
            _, conv, it, _ = mb.solve(tol=1e-30, max_iter=60, allow_noconv=True)
            runs.append(time.perf_counter() - t0)
            assert not conv and it == 60
        took[shift] = min(runs)
        mb.close()
    assert took[58.0] < 1.5 * took[20.0]


def test_an_undetermined_solution_is_found_out_before_the_iterations():
    """Too few states to connect the samples: the attempt with the inverse ends with the inverse
    (its iterations, up to 60 of them, were run first), and the solve goes on from f = 0."""
    t, mu = W.linear_grid(0.8046809556261122, 1.1828264986833577, 15), W.linear_grid(-7.0, -2.0, 2)
    mb, e, n, s = _loaded(t, mu, 115, 16, 90, 1.7399255687101833)
    f, conv, it, d = mb.solve(tol=1e-6, max_iter=10000)
    tried = mb.timing()[1] - it
    mb.close()
    beta, lnz = oracle.state_arrays(W.ideal_gas().replace(t=t, mu=mu, n_max=115))
    g, _ = oracle.mbar_iterate(beta, lnz, np.bincount(s, minlength=30), e, n, f)
    assert conv and np.max(np.abs(g - g[0] - f)) < 1e-6
    assert 0 < tried < 30


@pytest.mark.parametrize("n_mu", [32, 62, 63, 124])
def test_an_iteration_of_more_states_takes_little_longer(n_mu):
    """33 x 31 states (1023) against grids whose step holds more states per thread: the step's
    columns have to stay in registers."""
    per = []
    for m in (31, n_mu):
        t, mu = W.linear_grid(1.0, 1.6, 33), W.linear_grid(-3.6, -3.0, m)
        rng = np.random.default_rng(m)
        s = np.tile(np.arange(33 * m, dtype=np.int32), 20)
        n = rng.integers(10, 40, len(s)).astype(np.int32)
        mb = regc.Mbar(t, mu, 60)
        mb.set_samples(-0.5 * n + rng.normal(0.0, 1.0, len(s)), n, s)
        best = np.inf
        for _ in range(3):
            mb.solve(tol=1e-30, max_iter=40, allow_noconv=True)
            ms, it = mb.timing()
            best = min(best, ms / it)
        per.append(best)
        mb.close()
    assert per[1] < 4.0 * per[0]


@pytest.mark.parametrize("n_tgt,n_mu", [(1, 63), (2, 64), (3, 65), (1, 700)])
def test_targets_of_many_chemical_potentials(n_tgt, n_mu):
    """Groups of 64 chemical potentials and their remainders against the oracle, and the same
    values as one by one."""
    t, mu = W.linear_grid(1.0, 1.4, 4), W.linear_grid(-3.4, -3.0, 3)
    mb, e, n, s = _loaded(t, mu, 40, 100, 5)
    f, conv, _, _ = mb.solve(tol=1e-11)
    tt, tm = W.linear_grid(1.05, 1.35, n_tgt), W.linear_grid(-3.5, -2.9, n_mu)
    got, static = mb.targets(tt, tm), mb.targets_static(tt, tm)
    for k in (0, n_mu - 1):
        one = mb.targets(tt, tm[k: k + 1])
        for name in got:
            assert np.array_equal(got[name].reshape(n_tgt, n_mu, -1)[:, k], one[name].reshape(n_tgt, -1)), name
    mb.close()
    beta, lnz = oracle.state_arrays(W.ideal_gas().replace(t=t, mu=mu, n_max=40))
    _, logd = oracle.mbar_iterate(beta, lnz, np.bincount(s, minlength=12), e, n, f)
    ref = oracle.mbar_targets(np.repeat(1.0 / np.array(tt), n_mu),
                              np.array([oracle.state_lnz(a, b) for a in tt for b in tm]), e, n, logd, 40)
    assert conv
    for name in static:
        assert np.array_equal(static[name], got[name]), name
    assert np.allclose(got["mean_n"], ref["mean_n"], rtol=1e-8) and np.allclose(got["p_n"], ref["p_n"], atol=1e-10)
    assert np.array_equal(got["phase"], ref["phase"])


def test_many_chemical_potentials_take_no_longer_than_many_temperatures():
    """2 x 700 targets took 390 us in one block per temperature (350 x 4: 150)."""
    import time
    t, mu = W.linear_grid(1.0, 1.4, 4), W.linear_grid(-3.4, -3.0, 3)
    mb, *_ = _loaded(t, mu, 40, 100, 5)
    mb.solve(tol=1e-11)
    took = []
    for a, b in ((350, 4), (2, 700)):
        tt, tm = W.linear_grid(1.05, 1.35, a), W.linear_grid(-3.5, -2.9, b)
        runs = []
        for _ in range(20):
            t0 = time.perf_counter()
            mb.targets(tt, tm)
            runs.append(time.perf_counter() - t0)
        took.append(min(runs))
    mb.close()
    assert took[1] < 1.5 * took[0]


@pytest.mark.parametrize("burn,records", [(300, 100), (1000, 300)])
def test_samples_of_a_run_across_the_condensation(burn, records):
    """The sampler's own samples, energies of a gas and a liquid at the same N: at and beyond the
    exponents' limits.  The solution is a fixed point of the oracle's map and the averages at
    targets are the oracle's with it."""
    w = W.config2().replace(mu=W.linear_grid(-8.0, -2.0, 8), sample_every=10)
    with regc.Regc(w, precision=regc.FP32PAIR, sample_capacity=(burn // 10 + records) * w.n_states) as g:
        g.run(burn + 10 * records)
        e, n, s = (g.samples()[k][burn // 10 * w.n_states:] for k in ("e", "n", "state"))
    mb = regc.Mbar(w.t, w.mu, w.n_max)
    mb.set_samples(e, n, s)
    f, conv, it, d = mb.solve(tol=1e-8, max_iter=20000)
    assert conv and d < 1e-8
    beta, lnz = oracle.state_arrays(w)
    g, logd = oracle.mbar_iterate(beta, lnz, np.bincount(s, minlength=len(beta)), e, n, f)
    assert np.max(np.abs(g - g[0] - f)) < 1e-7
    tt, tm = W.linear_grid(0.45, 2.1, 9), W.linear_grid(-8.5, -1.5, 11)
    tz = np.array([oracle.state_lnz(T, u, w.lambda1) for T in tt for u in tm])
    ref = oracle.mbar_targets(np.repeat(1.0 / tt, len(tm)), tz, e, n, logd, w.n_max)
    got = mb.targets(tt, tm)
    # (log D is of the solution to some times its residual)
    assert np.allclose(got["mean_n"], ref["mean_n"], rtol=1e-6, atol=1e-6)
    assert np.allclose(got["mean_e"], ref["mean_e"], rtol=1e-6, atol=1e-6)
    mb.close()
