"""The chirp table of a beam carries the gain correction of the schedule that reads
it: in a single-launch plan of mixed lengths the mixed kernel runs a 4096-point beam
with another schedule than the beam's own call does by default.  The same schedule in
a one-shot call differs by FP32 rounding alone: below 1e-7 in each of 33,333 outputs,
so 6e-10 in their sum; 5e-9 allowed.  (The other schedule's correction would shift
the sum by 2.3e-8.)"""
import numpy as np
import pytest

from tests.test_gpu_parity import _beam_int8, _cdd
from tests.util import flush, to_dev

pytestmark = pytest.mark.gpu


def test_mixed_plan_reads_the_table_of_its_schedule():
    import torch
    cdd = _cdd()
    nchan, fcen, df, dm = 16, 330.0, 0.02, 20.0
    v = to_dev(_beam_int8(90, 100_000, nchan, fcen, df * nchan, dm))
    flush("case: 4096 points beside 2048 in one launch")
    plan = cdd.Plan([dict(voltages=v, f_centre=fcen, bw=df * nchan, dms=[dm], n_int=3, fft_len=n)
                     for n in (4096, 2048)], single_launch=True)
    plan.execute()
    torch.cuda.synchronize()
    info = plan.info(0)
    one = cdd.dedisperse(v, fcen, df * nchan, dm, 4096, 3, variant=3, overlap=info["overlap"],
                         nfront=info["nfront"])
    torch.cuda.synchronize()
    a = plan.I[0][0].double().sum().item()
    b = one["I"].double().sum().item()
    print("sum ratio - 1: %.2e" % (a / b - 1.0))
    assert abs(a / b - 1.0) <= 5e-9
    assert np.array_equal(plan.cov[0][0].cpu().numpy(), one["cov"].cpu().numpy())
    plan.close()
