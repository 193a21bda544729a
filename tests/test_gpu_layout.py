"""The layout change at the edges of its tiles, with the chirp table and the
channel delays written by the same kernel and (more channels than tiles) by
kernels of their own, against the FP64 oracle.  Tolerances as in
test_gpu_parity (relative L2 1e-5 on voltages, 1e-4 on intensities)."""
import numpy as np
import pytest

from tests.test_gpu_parity import _beam_int8, _check, _run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["int8", "complex64"])
@pytest.mark.parametrize("nchan,nsamp", [(2, 4100), (63, 2016), (64, 2048), (65, 2081), (129, 321),
                                         (200, 90), (500, 65)])
def test_layout_change(nchan, nsamp, kind):
    fcen, bw, dm = 610.0, 0.03125 * nchan, 12.0
    v = _beam_int8(300 + nchan, nsamp, nchan, fcen, bw, dm)
    if kind == "complex64":
        v = np.ascontiguousarray(v[..., 0] + 1j * v[..., 1]).astype(np.complex64)
    got, o, _ = _run_both(v, fcen, bw, dm, 1, 256)
    _check(got, o)
