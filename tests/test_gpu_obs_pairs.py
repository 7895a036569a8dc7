"""The structural observables of one configuration against plain FP64 counts: layers of no,
one, two, an odd and an even number of members, and of as many as the kernel keeps in LDS
(1024) and more."""
import numpy as np
import pytest

from paper_1908_11118_amd import regc
from paper_1908_11118_amd import workloads as W

pytestmark = pytest.mark.gpu

DZ, LAYER, DR, NR = 0.25, (1.0, 2.0), 0.05, 120


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def counts(w, x):
    nz = int(np.ceil((w.zhi - w.zlo) / DZ))
    k = np.clip(np.floor((x[:, 2] - w.zlo) / DZ).astype(int), 0, nz - 1)
    out = [np.bincount(k, minlength=nz)]
    m = x[(x[:, 2] >= LAYER[0]) & (x[:, 2] < LAYER[1])]
    d = m[:, None, :2] - m[None, :, :2]
    for q, box in enumerate((w.lx, w.ly)):
        d[..., q] = np.where(d[..., q] > 0.5 * box, d[..., q] - box, np.where(d[..., q] < -0.5 * box, d[..., q] + box, d[..., q]))
    i, j = np.triu_indices(len(m), 1)
    b = np.floor(np.sqrt(d[i, j, 0] * d[i, j, 0] + d[i, j, 1] * d[i, j, 1]) / DR).astype(int)
    out += [np.bincount(b[b < NR], minlength=NR), [len(m)]]
    return np.concatenate(out)


@pytest.mark.parametrize("members", [0, 1, 2, 7, 64, 255, 1024, 1025])
def test_counts_of_a_configuration(members):
    rng = np.random.default_rng(members)
    w = W.ideal_gas(n_t=1, n_mu=2, n_max=1100).replace(sample_every=1, trials_per_sweep=1)
    g = regc.Regc(w, precision=regc.FP64, sample_capacity=8)
    g.set_observables(DZ, LAYER, DR, NR)
    start = []
    for _ in range(2):
        x = rng.random((members + 5, 3)) * [w.lx, w.ly, 1.0] + [0.0, 0.0, 1.0]
        x[members:, 2] = rng.random(5) * 0.9
        start.append(x)
    g.set_walkers([members + 5] * 2, start)
    g.run(1)
    got, now = g.observables(), g.walkers()
    g.close()
    for k in range(2):
        ref = counts(w, now["xyz"][k, : now["n"][k]])
        assert np.array_equal(got[k][: len(ref)], ref)
