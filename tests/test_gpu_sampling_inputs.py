"""Sampling where an input leaves the usual range: slab atoms given outside the cell, an
acceptance threshold that overflows, pair terms that do, runs of more pairs than 32 bits count, molecular dynamics that blows up, a particle at the edge of the slab's reach."""
import numpy as np
import pytest

import oracle
from paper_1908_11118_amd import regc
from paper_1908_11118_amd import workloads as W

pytestmark = pytest.mark.gpu
ACC, CORE = [1, 3, 5], 9                  # accepted moves by kind, hard-core rejections


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    torch.cuda.set_device(0)


def _slab_system(cells, slab=None):
    box = 1.5 * cells
    slab = W.fcc100_slab(cells, 3, box, rc=2.5) if slab is None else slab
    return W.Workload(name="slab", slab=slab, lx=box, ly=box, zlo=0.0, zhi=7.0, t=np.array([0.8, 1.2]),
                      mu=np.array([-3.0, -2.5]), n_max=90)


def _run(w, precision, counts=(40, 50, 60, 70), sweeps=12, **kw):
    rng = np.random.default_rng(3)
    xyz = [W.random_configuration(rng, w, n) for n in counts]
    with regc.Regc(w, precision=precision, **kw) as g:
        g.set_walkers(list(counts), xyz)
        e0 = g.energies()
        g.run(sweeps)
        return e0, g.walkers(), g.stats()["stats"]


# 8 cells: columns; 4 cells: one list of all atoms.  Each atom by its own number of whole
# cells; every coordinate and box is a multiple of 0.75, so the shift is exact
@pytest.mark.parametrize("precision", [regc.FP32PAIR, regc.FP64])
@pytest.mark.parametrize("cells", [4, 8])
@pytest.mark.parametrize("away", [(-2, -2), (2, 3), (-3, -2, 0, 2)])
def test_slab_atoms_whole_cells_away(precision, cells, away):
    w = _slab_system(cells)
    slab = w.slab.copy()
    slab[:, :2] += w.lx * np.random.default_rng(5).choice(away, (len(slab), 2))
    a, b = _run(w, precision), _run(_slab_system(cells, slab), precision)
    assert np.array_equal(a[0], b[0])
    assert np.array_equal(a[2], b[2])
    for name in ("n", "e", "xyz"):
        assert np.array_equal(a[1][name], b[1][name]), name


# (a coordinate within half a cell of the cell is rounded where it lies: about 1e-6 in FP32, times
# a slope of at most 400 at the distances of these configurations, over some 60 close pairs)
@pytest.mark.parametrize("precision,tol", [(regc.FP32PAIR, 0.05), (regc.FP64, 1e-9)])
@pytest.mark.parametrize("cells", [4, 8])
@pytest.mark.parametrize("away", [-1, 1])
def test_energies_with_the_slab_in_the_next_cell(precision, tol, cells, away):
    w = _slab_system(cells)
    slab = w.slab.copy()
    slab[:, :2] += away * w.lx
    a, b = _run(w, precision, sweeps=0), _run(_slab_system(cells, slab), precision, sweeps=0)
    assert np.allclose(a[0], b[0], rtol=0, atol=tol)


@pytest.mark.parametrize("cells", [4, 8])
def test_slab_atoms_within_half_a_cell_are_taken_as_given(cells):
    """A slab centred on the cell's corner: FP64 trajectories are the oracle's, which reads
    the coordinates as they are."""
    w = _slab_system(cells)
    slab = w.slab.copy()
    slab[:, :2] -= np.where(slab[:, :2] > 0.5 * w.lx, w.lx, 0.0)
    slab[::7, 0] += 0.1
    w = _slab_system(cells, slab)
    rng = np.random.default_rng(3)
    counts = [40, 50, 60, 70]
    xyz = [W.random_configuration(rng, w, n) for n in counts]
    x = np.zeros((4, w.n_max, 3))
    for k in range(4):
        x[k, : counts[k]] = xyz[k]
    ref = oracle.Chain(w)
    ref.set_walkers(counts, x)
    r = ref.run(6, trace=True)
    with regc.Regc(w, precision=regc.FP64, trace_capacity=6) as g:
        g.set_walkers(counts, xyz)
        g.run(6)
        bits, _ = g.trace(6)
        wk = g.walkers()
    assert np.array_equal(bits, r["bits"])
    assert np.allclose(wk["e"], ref.e, rtol=1e-10, atol=1e-9)


@pytest.mark.parametrize("precision", [regc.FP32PAIR, regc.FP64])
@pytest.mark.parametrize("split", [1, 2, 4])
def test_hard_core_under_an_infinite_threshold(precision, split):
    """T = 1e308: (ln prefactor - ln U) T overflows, and still no pair comes closer than the
    hard core."""
    w = W.small_lj(n_t=1, n_mu=1, n_max=40).replace(t=np.array([1e308]), mu=np.array([0.0]), hc_frac=0.9)
    with regc.Regc(w, precision=precision, split=split, walkers_per_block=1) as g:
        g.run(8)
        wk, st = g.walkers(), g.stats()["stats"]
    x = wk["xyz"][0, : wk["n"][0]]
    d = x[:, None] - x[None]
    d[..., :2] -= np.array([w.lx, w.ly]) * np.rint(d[..., :2] / np.array([w.lx, w.ly]))
    r = np.sqrt((d ** 2).sum(-1))[np.triu_indices(len(x), 1)]
    assert len(x) > 5 and st[0, CORE] > 0
    assert r.min() >= 0.9 * w.sig_gg * (1 - 1e-6)


@pytest.mark.parametrize("split", [1, 2, 4])
def test_infinite_pair_terms_are_not_hard_cores(split):
    """Without a hard core a pair term past FP32's range is an ordinary rejection."""
    w = W.small_lj(n_t=1, n_mu=1, n_max=40).replace(t=np.array([1.0]), mu=np.array([4.0]), hc_frac=0.0, sig_gg=1e5,
                                                    shifted=0, slab=np.zeros((0, 3)))
    with regc.Regc(w, precision=regc.FP32PAIR, split=split, walkers_per_block=1) as g:
        g.run(20)
        wk, st = g.walkers(), g.stats()["stats"]
    att, acc = st[0, [0, 2, 4]].sum(), st[0, ACC].sum()
    assert wk["n"][0] > 0 and att > acc + st[0, [6, 7, 8]].sum()      # some were rejected on their energy
    assert st[0, CORE] == 0


@pytest.mark.parametrize("per,sweeps", [(1000, 1000), (1000000, 1)])
def test_pairs_past_32_bits(per, sweeps):
    """4000 particles in a layer two cutoffs wide, a million displacements in one call, of
    many sweeps or of a single one: about 5e9 pairs inside the cutoff, and their share of the
    candidates is that of a short run."""
    n = 4000
    w = W.Workload(name="pairs", slab=np.zeros((0, 3)), lx=5.0, ly=5.0, zlo=0.0, zhi=0.01, t=np.array([1.0]),
                   mu=np.array([0.0]), n_max=n, eps_gg=0.0, sig_gg=1e-3, hc_frac=0.0, p_disp=1.0, p_ins=0.0,
                   trials_per_sweep=per, max_disp=0.004, swap_every=0, sample_every=0)
    x = np.random.default_rng(1).random((n, 3)) * [5.0, 5.0, 0.01]
    share = []
    for k, system in ((5, w.replace(trials_per_sweep=1000)), (sweeps, w)):
        with regc.Regc(system, precision=regc.FP32PAIR, split=1, walkers_per_block=1, sweeps_per_launch=k) as g:
            g.set_walkers([n], [x])
            g.run(k)
            cand, useful = g.pair_counts()
        share.append(useful / cand)
    assert 2 ** 32 < useful < cand
    assert abs(share[1] - share[0]) < 0.02


def test_md_that_blows_up_reports_it():
    """An infinite time step: positions and energy are not numbers, in the oracle as here."""
    w = W.small_lj(n_t=1, n_mu=1, n_max=10).replace(schedule=1, x0=0.0, md_steps=1, md_dt=float("inf"), sample_every=1)
    x = W.random_configuration(np.random.default_rng(2), w, 6)
    ref = oracle.Chain(w)
    full = np.zeros((1, 10, 3))
    full[0, :6] = x
    ref.set_walkers([6], full)
    ref.run(1)
    with regc.Regc(w, precision=regc.FP64) as g:
        g.set_walkers([6], [x])
        g.run(1)
        e = g.walkers(xyz=False)["e"][0]
    assert np.isnan(ref.e[0]) and np.isnan(e)


@pytest.mark.parametrize("precision", [regc.FP32PAIR, regc.FP64])
def test_md_at_the_edge_of_the_slabs_reach(precision):
    """A particle right above the slab's atom, closer than the cutoff by less than FP32
    resolves the cutoff (2.6 in FP32 is 2.5999999)."""
    z = float(np.float32(2.6))
    w = W.Workload(name="edge", slab=np.array([[3.0, 3.0, 0.0]]), lx=6.0, ly=6.0, zlo=0.5, zhi=5.0, t=np.array([1.0]),
                   mu=np.array([-3.0]), n_max=4, rc=2.6, shifted=0, schedule=1, x0=0.0, md_steps=1, md_dt=1e-30,
                   md_tau=0.0, sample_every=1)
    with regc.Regc(w, precision=precision) as g:
        g.set_walkers([1], [np.array([[3.0, 3.0, z]])])
        g.run(1)
        e = g.walkers(xyz=False)["e"][0]
    c6 = z ** -6
    assert e == pytest.approx(4.0 * (c6 * c6 - c6), rel=1e-5)
