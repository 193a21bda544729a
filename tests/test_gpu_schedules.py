"""Every compiled schedule of the block kernels against the FP64 oracle: each
has its own twiddle tables and its own layout of the chirp table (both paired
by the radices of its passes).  Tolerances as in test_gpu_parity (relative L2
1e-5 on voltages, 1e-4 on intensities): FP32 transforms of these lengths stay
an order of magnitude below them."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import TOL_I, _beam_int8, _cdd, _check, _run_both
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu

SCHEDULES = [(256, 0), (512, 0), (1024, 0), (2048, 0)] + [(4096, v) for v in range(4)] + \
    [(8192, v) for v in range(10)] + [(16384, v) for v in range(4)]


@pytest.mark.parametrize("kind", ["int8", "complex64"])
@pytest.mark.parametrize("N,variant", SCHEDULES)
def test_schedule_against_oracle(N, variant, kind):
    nchan, fcen, df, dm = 3, 330.0, 0.02, 25.0
    v = _beam_int8(700 + N + variant, N + N // 2 + 5, nchan, fcen, df * nchan, dm)
    if kind == "complex64":
        v = np.ascontiguousarray(v[..., 0] + 1j * v[..., 1]).astype(np.complex64)
    got, o, info = _run_both(v, fcen, df * nchan, dm, 3, N, taper="hann", variant=variant)
    assert info["fft_len"] == N
    _check(got, o)


@pytest.mark.parametrize("single_launch", [False, True])
@pytest.mark.parametrize("N,variant", [(8192, 4), (8192, 1), (16384, 2), (4096, 2)])
def test_chirp_table_of_a_plan_fits_the_kernel_that_reads_it(N, variant, single_launch):
    """A one-DM plan with a schedule asked for: one launch per beam runs that
    schedule, the single-launch form the default one; the table follows."""
    import torch
    cdd = _cdd()
    nchan, fcen, df, dm = 4, 330.0, 0.02, 25.0
    flush("case: plan N=%d variant=%d single_launch=%s" % (N, variant, single_launch))
    raw = [_beam_int8(900 + N + k, 2 * N + 17 * k, nchan, fcen, df * nchan, dm) for k in range(2)]
    plan = cdd.Plan([dict(voltages=to_dev(v), f_centre=fcen, bw=df * nchan, dms=[dm], n_int=4,
                          fft_len=N) for v in raw], variant=variant,
                    single_launch=single_launch)
    plan.execute()
    torch.cuda.synchronize()
    for b, v in enumerate(raw):
        info = plan.info(b)
        o = O.dedisperse(v, fcen, df * nchan, dm, 4, fft_len=N, overlap=info["overlap"],
                         nfront=info["nfront"])
        assert rel_l2(plan.I[b][0].cpu().numpy(), o["I"]) <= TOL_I
    plan.close()


@pytest.mark.parametrize("N", [4096, 8192, 16384])
@pytest.mark.parametrize("offset,nsamp_odd,overlap", [(0, 0, 256), (1, 0, 256), (0, 1, 256),
                                                      (1, 1, 255), (0, 0, 255)])
def test_first_pass_on_the_matrix_cores_at_any_alignment(N, offset, nsamp_odd, overlap):
    """Full-scale bytes in one channel, read in place: records on and off a
    4-byte boundary, of odd and even length, with blocks starting on odd
    samples (odd step), the last block cut short."""
    import torch
    cdd = _cdd()
    rng = np.random.default_rng(N + 10 * offset + nsamp_odd)
    nsamp = 2 * N + 100 + nsamp_odd
    v = rng.choice(np.array([-128, -1, 0, 1, 127], dtype=np.int8), size=(nsamp, 1, 2))
    buf = torch.zeros(2 * (nsamp + 8), dtype=torch.int8, device="cuda")
    buf[2 * offset:2 * offset + v.size] = to_dev(v).reshape(-1)
    d = buf[2 * offset:2 * offset + v.size].view(nsamp, 1, 2)
    flush("case: matrix first pass N=%d offset=%d nsamp=%d overlap=%d" % (N, offset, nsamp, overlap))
    g = cdd.dedisperse(d, 330.0, 0.02, 5.0, N, 1, want_chan=True, want_voltages=True,
                       overlap=overlap, nfront=128)
    torch.cuda.synchronize()
    o = O.dedisperse(v, 330.0, 0.02, 5.0, 1, fft_len=N, overlap=overlap, nfront=128,
                     want_voltages=True)
    _check({k: g[k].cpu().numpy() for k in ("I", "cov", "P", "y")}, o)
