"""FP64 trajectories against the oracle where the trial kernel's layout of the slab and
of the gas blocks changes: the slab in LDS with its periodic halo, without room for one
and unbinned; particle counts on both sides of a block of 64; a move mix whose
displacement threshold is the whole range of a random word."""
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


def _system(cells, n_max, **kw):
    box = 1.5 * cells
    return W.Workload(name="layout", slab=W.fcc100_slab(cells, 3, box, rc=2.5), lx=box, ly=box, zlo=0.0, zhi=9.0,
                      t=np.array([0.9, 1.6]), mu=np.array([-3.0, -2.0]), n_max=n_max, trials_per_sweep=70, **kw)


# 12 x 12 x 3 atoms in 6 x 6 columns: 13.8 KB in FP64 and 24.6 KB with the halo; 3600
# particles (144 KB with their ln k table) leave 160 KB no room for the second
@pytest.mark.parametrize("cells,n_max,split", [(12, 300, 1), (12, 300, 2), (12, 3600, 1), (12, 3600, 2), (4, 300, 1),
                                               (6, 300, 4)])
@pytest.mark.parametrize("p_disp", [0.5, 1.0])
def test_fp64_slab_layouts_and_block_edges(cells, n_max, split, p_disp):
    w = _system(cells, n_max, p_disp=p_disp, p_ins=0.5 * (1.0 - p_disp))
    rng = np.random.default_rng(cells)
    counts = [63, 64, 65, 129] if cells > 4 else [31, 32, 33, 20]
    xyz = [W.random_configuration(rng, w, n) for n in counts]
    x = np.zeros((4, n_max, 3))
    for k in range(4):
        x[k, : counts[k]] = xyz[k]
    ref = oracle.Chain(w)
    ref.set_walkers(counts, x)
    r = ref.run(4, trace=True)
    with regc.Regc(w, precision=regc.FP64, trace_capacity=4, split=split, walkers_per_block=1) as g:
        g.set_walkers(counts, xyz)
        g.run(4)
        bits, nps = g.trace(4)
        wk, st = g.walkers(), g.stats()["stats"]
    assert np.array_equal(bits, r["bits"]) and np.array_equal(nps, r["trace_n"])
    assert np.array_equal(st, ref.stats)
    assert np.allclose(wk["e"], ref.e, rtol=1e-10, atol=1e-9)
    for k in range(4):
        assert np.array_equal(wk["xyz"][k, : ref.n[k]], ref.xyz[k, : ref.n[k]])
