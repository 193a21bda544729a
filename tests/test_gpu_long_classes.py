"""Three-level long transforms that run their middle passes over several items or
over slices of the column classes, against the same results in 64 bits
(perf/cases.py): the full band with the chirp read from the call's table (records of
more than four blocks), and channels of several blocks.  Tolerances as in
test_gpu_parity; a class or a row in the wrong place is an error of the order of 1."""
import pytest

from perf import cases
from tests.test_gpu_parity import TOL_I, TOL_V, _cdd
from tests.util import flush

pytestmark = pytest.mark.gpu


def _rel(got, want):
    import torch
    got, want = got.to(want.device), want.reshape(-1)
    d = torch.linalg.vector_norm(got.reshape(-1).to(want.dtype) - want)
    return (d / torch.linalg.vector_norm(want)).item()


@pytest.mark.parametrize("lg,nchan,volt", [(24, 512, True), (25, 1024, False), (26, 2048, False)])
def test_full_band_table_with_three_levels(lg, nchan, volt):
    import torch
    cdd = _cdd()
    q = cdd.fullband_query(1 << 12, nchan, 610.0, 16.0, 1.0, 16, 1 << lg)
    nspec = 4 * q["step"] // (2 * nchan) + 1001
    case = dict(kind="fullband", f=610.0, bw=16.0, nchan=nchan, nspec=nspec, dm=1.0,
                fft_len=1 << lg, n_int=16, taper="hann", volt=volt)
    flush("case: full band, five blocks of 2^%d points" % lg)
    s = cases.prepare(case, lg)
    got = cases.run(s)
    torch.cuda.synchronize()
    assert cdd.fullband_query(nspec, nchan, 610.0, 16.0, 1.0, 16, 1 << lg)["nblocks"] == 5
    want = cases.exact(case, lg)
    assert _rel(got["I"], want["I"]) <= TOL_I
    if volt:
        assert _rel(got["y"], want["y"]) <= TOL_V


@pytest.mark.parametrize("lg,nchan,blocks,dtype,volt", [
    (23, 2, 3, "int8", False), (23, 1, 5, "complex64", True), (24, 1, 3, "complex64", False),
    (25, 1, 2, "int8", False)])
def test_channels_of_several_blocks(lg, nchan, blocks, dtype, volt):
    import torch
    cdd = _cdd()
    f, bw, dm, N = 610.0, 16.0 * nchan, 1.0, 1 << lg
    dt = cdd.CDD_CI8 if dtype == "int8" else cdd.CDD_CF32
    q = cdd.query(dt, 1 << 12, nchan, f, bw, dm, N, 16)
    nsamp = (blocks - 1) * q["step"] + 100_001
    case = cases._beam("", f, bw, nchan, nsamp, dm, N, 16, dtype, "none", volt, nchan > 1)
    assert cdd.query(dt, nsamp, nchan, f, bw, dm, N, 16)["nblocks"] == blocks
    flush("case: %d channels, %d blocks of 2^%d points" % (nchan, blocks, lg))
    s = cases.prepare(case, lg)
    got = cases.run(s)
    torch.cuda.synchronize()
    want = cases.exact(case, lg)
    for k in ("I", "P"):
        if k in want:
            assert _rel(got[k], want[k]) <= TOL_I
    if volt:
        assert _rel(got["y"], want["y"]) <= TOL_V
