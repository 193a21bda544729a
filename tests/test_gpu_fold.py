"""Folding with a workgroup, a wave and a thread per bin, against the FP64
oracle: counts exact, the sums, formed in FP64, within one FP32 rounding (6e-8)."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import _cdd
from tests.util import flush, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins", [1, 7, 256, 1024, 1025, 8192, 8193])
@pytest.mark.parametrize("t_int,period,phase0", [
    (1, 10.0, 0.0), (5000, 1.5, 0.3), (20011, 1390.625, -2.75), (4096, 64.0, 0.5),
    (300, 5000.0, 7.25)])
def test_fold_layouts(nbins, t_int, period, phase0):
    import torch
    cdd = _cdd()
    flush("case: fold nbins=%d t_int=%d period=%g phase0=%g" % (nbins, t_int, period, phase0))
    x = np.random.default_rng(nbins + t_int).standard_normal(t_int).astype(np.float32)
    prof, cnt = cdd.fold(to_dev(x), period, phase0, nbins)
    torch.cuda.synchronize()
    op, oc = O.fold(x.astype(np.float64), period, phase0, nbins)
    assert np.array_equal(cnt.cpu().numpy(), oc)
    assert np.abs(prof.cpu().numpy() - op).max() <= 6e-8 * max(1.0, np.abs(op).max())
