"""What the getters return against plain copies of the device arrays, below and above the size
up to which they are packed into pinned memory (256 KiB: 16 384 samples of 16 bytes), whole
and with pieces left out."""
import ctypes as C

import numpy as np
import pytest

from paper_1908_11118_amd import regc
from paper_1908_11118_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("records", [0, 1, 1023, 1024, 1025, 5000])
def test_samples_are_the_device_arrays(records):
    import torch
    w = W.ideal_gas(n_t=4, n_mu=4, n_max=6).replace(sample_every=1)
    g = regc.Regc(w, sample_capacity=16 * max(records, 1) + 16)
    g.run(records)
    got = g.samples()
    ptr = [C.c_void_p() for _ in range(3)]
    cnt = C.c_int64()
    regc.lib().regc_samples_device(g.h, *[C.byref(p) for p in ptr], C.byref(cnt))
    assert cnt.value == 16 * records == len(got["e"])
    torch.cuda.synchronize()
    hip = C.CDLL("libamdhip64.so")
    for p, name, dtype in zip(ptr, ("e", "n", "state"), (np.float64, np.int32, np.int32)):
        ref = np.zeros(cnt.value, dtype)
        if cnt.value:
            assert hip.hipMemcpy(ref.ctypes.data_as(C.c_void_p), p, C.c_size_t(ref.nbytes), 2) == 0
        assert np.array_equal(got[name], ref)
    n_only = np.zeros(cnt.value, np.int32)
    have = C.c_int64()
    regc.lib().regc_get_samples(g.h, None, n_only.ctypes.data_as(C.POINTER(C.c_int32)), None, cnt.value, C.byref(have))
    assert have.value == cnt.value and np.array_equal(n_only, got["n"])
    x, light = g.walkers(), g.walkers(xyz=False)
    for name in ("n", "e", "label"):
        assert np.array_equal(x[name], light[name])
    for k in range(16):
        inside = x["xyz"][k, : x["n"][k]]
        assert np.all(inside[:, :2] >= 0) and np.all(x["xyz"][k, x["n"][k]:] == 0)
    g.close()
