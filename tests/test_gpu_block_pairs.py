"""DM trials in workgroups of two neighbouring blocks of a channel, with a spare
group at the end of every channel (nine blocks each, more of them than compute
units), against the FP64 oracle; tolerance as in test_gpu_parity."""
import pytest

import oracle as O
from tests.test_gpu_block_groups import _signal
from tests.test_gpu_parity import TOL_I, _cdd
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["int8", "complex64"])
@pytest.mark.parametrize("dms", [[20.0, 21.5, 23.0], [20.0, 20.4, 23.0]], ids=["even", "uneven"])
@pytest.mark.parametrize("N", [512, 1024, 2048, 4096])
def test_trials_of_two_blocks_and_a_spare_one(N, dms, kind):
    import torch
    cdd = _cdd()
    nchan, fcen, df = 40, 330.0, 0.02
    step = cdd.query(cdd.CDD_CI8, N, nchan, fcen, df * nchan, dms[-1], N, 2)["step"]
    v = _signal(70 + N, 8 * step + step // 3, nchan, fcen, df * nchan, 22.0, kind)
    flush("case: nine blocks, N=%d %s %s" % (N, dms, kind))
    plan = cdd.Plan([dict(voltages=to_dev(v), f_centre=fcen, bw=df * nchan, dms=dms, n_int=2,
                          fft_len=N)])
    plan.execute()
    torch.cuda.synchronize()
    info = plan.info(0)
    assert info["nblocks"] == 9
    for i, dm in enumerate(dms):
        o = O.dedisperse(v, fcen, df * nchan, dm, 2, fft_len=N, overlap=info["overlap"],
                         nfront=info["nfront"])
        assert rel_l2(plan.I[0][i].cpu().numpy(), o["I"]) <= TOL_I
    plan.close()
