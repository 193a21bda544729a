"""Detection straight from the record with integrations above 16 samples, in records
short or large enough for that form, against the FP64 oracle.  Bounds as in test_gpu_detect: int8 sums are whole numbers below 2^24, so P
is exact; float sums are within n_int FP32 roundings, the aligned sum within nchan
more."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import _cdd
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nchan,nsamp,n_int,kind", [
    (67, 17 * 33 + 1, 17, "int8"), (64, 20 * 33, 20, "int8"), (3, 31 * 6500, 31, "int8"),
    (130, 24 * 970 + 5, 24, "int8"), (132, 64 * 712 + 9, 64, "int8"), (8, 40 * 9, 40, "int8"),
    (3, 17 * 11800 + 1, 17, "complex64"), (65, 32 * 1450, 32, "complex64"),
    (100, 63 * 960, 63, "complex64"), (7, 48 * 10, 48, "complex64")])
def test_long_integrations_from_the_record(nchan, nsamp, n_int, kind):
    import torch
    cdd = _cdd()
    flush("case: incoherent %s nchan=%d nsamp=%d n_int=%d" % (kind, nchan, nsamp, n_int))
    rng = np.random.default_rng(1000 * nchan + n_int)
    if kind == "int8":
        v = rng.integers(-128, 128, size=(nsamp, nchan, 2)).astype(np.int8)
    else:
        v = (rng.standard_normal((nsamp, nchan)) +
             1j * rng.standard_normal((nsamp, nchan))).astype(np.complex64)
    bw = nchan * 0.0625
    g = cdd.incoherent(to_dev(v), 325.0, bw, 5.0, n_int, want_chan=True)
    torch.cuda.synchronize()
    o = O.incoherent(v, 325.0, bw, 5.0, n_int)
    P = g["P"].cpu().numpy()
    if kind == "int8":
        assert np.array_equal(P, o["P"])
    else:
        assert rel_l2(P, o["P"]) <= n_int * 6e-8
    assert rel_l2(g["I"].cpu().numpy(), o["I"]) <= (n_int + nchan) * 6e-8
    assert np.array_equal(g["cov"].cpu().numpy(), o["cov"])
