"""Detection straight from the time-major record, at the edges of its tiles,
against the FP64 oracle.

Intensities: int8 sums are whole numbers below 2^24, so P is exact; float sums
of n_int terms are within n_int FP32 roundings (n_int 6e-8 relative), the
aligned sum within nchan more."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import _cdd
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["int8", "complex64"])
@pytest.mark.parametrize("nchan,nsamp,n_int", [
    (2, 40, 1), (3, 31, 1), (4, 33 * 2, 2), (63, 700, 3), (64, 32 * 4, 4), (65, 33 * 4 + 3, 4),
    (128, 1000, 8), (130, 777, 5), (132, 64 * 40 + 1, 64), (132, 65 * 9, 65), (260, 300, 16)])
def test_incoherent_tiles(nchan, nsamp, n_int, kind):
    import torch
    cdd = _cdd()
    flush("case: incoherent %s nchan=%d nsamp=%d n_int=%d" % (kind, nchan, nsamp, n_int))
    rng = np.random.default_rng(1000 * nchan + n_int)
    v = rng.integers(-128, 128, size=(nsamp, nchan, 2)).astype(np.int8)
    if kind == "complex64":
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


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_incoherent_record_off_an_eight_byte_boundary(offset):
    """A record that starts on any 2-byte boundary (a view into a longer one)."""
    import torch
    cdd = _cdd()
    rng = np.random.default_rng(offset)
    v = rng.integers(-128, 128, size=(500, 8, 2)).astype(np.int8)
    buf = torch.zeros(v.size + 64, dtype=torch.int8, device="cuda")
    buf[2 * offset:2 * offset + v.size] = to_dev(v).reshape(-1)
    d = buf[2 * offset:2 * offset + v.size].view(500, 8, 2)
    flush("case: incoherent at byte offset %d" % (2 * offset))
    g = cdd.incoherent(d, 325.0, 0.5, 5.0, 4, want_chan=True)
    torch.cuda.synchronize()
    assert np.array_equal(g["P"].cpu().numpy(), O.incoherent(v, 325.0, 0.5, 5.0, 4)["P"])
