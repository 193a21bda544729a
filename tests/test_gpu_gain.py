"""Mean gain of the transforms: the sum of the intensities against the FP64 oracle.

Rounding errors of the data average out in a sum of 100,000 outputs (below 1e-9);
what is left is the loss that the rounding of constants and twiddles causes alike in
every sample, 1.5e-7 to 6.6e-7, and its correction in the chirp.  Allowed is a third
of an FP32 rounding (2^-24 = 6e-8) for a channel's transforms and half of one for the
full band, whose records are transformed back first: a correction of the wrong size,
or one applied after its factors are rounded (2 to 9e-8), does not pass."""
import numpy as np
import pytest

import oracle as O
import synth
from tests.test_gpu_parity import _cdd
from tests.util import flush, to_dev

pytestmark = pytest.mark.gpu
TOL, TOL_BAND = 2e-8, 3e-8


def _record(nsamp, nchan, kind, seed):
    v = np.random.default_rng(seed).integers(-60, 61, size=(nsamp, nchan, 2), dtype=np.int8)
    return v if kind == "int8" else np.ascontiguousarray(
        v.astype(np.float32)).view(np.complex64)[..., 0]


def _shift(got, want):
    s = got.double().sum().item() / np.sum(want, dtype=np.float64) - 1.0
    print("shift of the sum: %+.2e" % s, flush=True)
    return abs(s)


@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096, 8192, 16384])
@pytest.mark.parametrize("kind", ["int8", "complex64"])
def test_one_dm(kind, N):
    import torch
    cdd = _cdd()
    v = _record(200_000, 2, kind, N)
    dm = 5.0 if N < 2048 else 30.0
    flush("case: gain at %d points, %s" % (N, kind))
    g = cdd.dedisperse(to_dev(v), 325.0, 0.125, dm, N, 4)
    torch.cuda.synchronize()
    o = O.dedisperse(v, 325.0, 0.125, dm, 4, fft_len=N, overlap=g["info"]["overlap"],
                     nfront=g["info"]["nfront"])
    assert _shift(g["I"], o["I"]) <= TOL


@pytest.mark.parametrize("dms", [[5.0, 5.1, 5.2], [5.0, 5.13, 5.2]], ids=["even", "uneven"])
@pytest.mark.parametrize("kind,N", [("complex64", n) for n in (512, 1024, 2048, 4096, 8192, 16384)]
                         + [("int8", n) for n in (4096, 8192, 16384)])
def test_trials(kind, N, dms):
    import torch
    cdd = _cdd()
    v = _record(200_000, 2, kind, N + 1)
    flush("case: gain of trials %s at %d points, %s" % (dms, N, kind))
    plan = cdd.Plan([dict(voltages=to_dev(v), f_centre=325.0, bw=0.125, dms=dms, n_int=4)],
                    fft_len=N)
    plan.execute()
    torch.cuda.synchronize()
    info = plan.info(0)
    for i in (0, 1):
        o = O.dedisperse(v, 325.0, 0.125, dms[i], 4, fft_len=N, overlap=info["overlap"],
                         nfront=info["nfront"])
        assert _shift(plan.I[0][i], o["I"]) <= TOL
    plan.close()


@pytest.mark.parametrize("lg", [15, 17, 18, 20, 23])
def test_long_transforms(lg):
    import torch
    cdd = _cdd()
    v = _record(max(3 << (lg - 1), 1 << 20), 1, "complex64", lg)[:, 0]
    flush("case: gain at 2^%d points" % lg)
    g = cdd.dedisperse(to_dev(v), 610.0, 16.0, 1.0, 1 << lg, 16)
    torch.cuda.synchronize()
    o = O.dedisperse(v[:, None], 610.0, 16.0, 1.0, 16, fft_len=1 << lg,
                     overlap=g["info"]["overlap"], nfront=g["info"]["nfront"])
    assert _shift(g["I"], o["I"]) <= TOL


@pytest.mark.parametrize("nchan,lg", [(512, 16), (128, 16), (512, 19), (2048, 20)])
def test_full_band(nchan, lg):
    import torch
    cdd = _cdd()
    sp = synth.noise_int8(synth.rng_for(6, salt=lg), (1 << 21) // nchan, nchan, 20.0)
    flush("case: gain of the full band, %d bins, 2^%d points" % (nchan, lg))
    g = cdd.fullband(to_dev(sp), 610.0, 16.0, 1.0, 16, 1 << lg)
    torch.cuda.synchronize()
    o = O.fullband_dedisperse(sp, 610.0, 16.0, 1.0, 16, fft_len=1 << lg,
                              overlap=g["info"]["overlap"], nfront=g["info"]["nfront"])
    assert _shift(g["I"], o["P"]) <= TOL_BAND
