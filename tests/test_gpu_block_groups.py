"""Workgroups that hold several blocks of one channel (four at 256 points, two
of a DM tile up to 4096 points): block counts per channel that leave groups of
the last workgroup idle, against the FP64 oracle.  Tolerances as in
test_gpu_parity (relative L2 1e-5 on voltages, 1e-4 on intensities)."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import TOL_I, _beam_int8, _cdd, _check, _run_both
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu


def _signal(seed, nsamp, nchan, fcen, bw, dm, kind):
    v = _beam_int8(seed, nsamp, nchan, fcen, bw, dm)
    if kind == "complex64":
        v = np.ascontiguousarray(v[..., 0] + 1j * v[..., 1]).astype(np.complex64)
    return v


@pytest.mark.parametrize("kind", ["int8", "complex64"])
@pytest.mark.parametrize("nsamp", [90, 300, 700, 811, 1001, 2003])
def test_short_blocks_fill_a_wave(nsamp, kind):
    nchan, fcen, df, dm = 3, 330.0, 0.02, 9.0
    v = _signal(40 + nsamp, nsamp, nchan, fcen, df * nchan, dm, kind)
    got, o, info = _run_both(v, fcen, df * nchan, dm, 2, 256)
    assert info["fft_len"] == 256
    _check(got, o)


@pytest.mark.parametrize("single_launch", [False, True])
@pytest.mark.parametrize("kind", ["int8", "complex64"])
@pytest.mark.parametrize("dms", [[20.0, 21.5, 23.0, 24.5], [20.0, 20.4, 23.0]],
                         ids=["even", "uneven"])
@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096])
def test_trials_of_neighbouring_blocks(N, dms, kind, single_launch):
    """One, two, three and five blocks a channel in one plan."""
    import torch
    cdd = _cdd()
    nchan, fcen, df = 3, 330.0, 0.02
    raw = [_signal(60 + N + int(4 * m), int(m * N), nchan, fcen, df * nchan, 22.0, kind)
           for m in (0.5, 1.5, 2.25, 3.75)]
    flush("case: trials N=%d %s %s single_launch=%s" % (N, dms, kind, single_launch))
    plan = cdd.Plan([dict(voltages=to_dev(v), f_centre=fcen, bw=df * nchan, dms=dms, n_int=2,
                          fft_len=N) for v in raw], single_launch=single_launch)
    plan.execute()
    torch.cuda.synchronize()
    for b, v in enumerate(raw):
        info = plan.info(b)
        for i, dm in enumerate(dms):
            o = O.dedisperse(v, fcen, df * nchan, dm, 2, fft_len=N, overlap=info["overlap"],
                             nfront=info["nfront"])
            assert rel_l2(plan.I[b][i].cpu().numpy(), o["I"]) <= TOL_I
    plan.close()


@pytest.mark.parametrize("nfront", [32, 30])
@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096, 8192, 16384])
def test_sums_of_four(N, nfront):
    """n_int 4 with a leading overlap that is a multiple of four samples (sums
    between lanes) and one that is not (through LDS); a record that ends inside
    a block, stored and accumulated."""
    import torch
    cdd = _cdd()
    nchan, fcen, df, dm = 3, 330.0, 0.02, 6.0
    v = _beam_int8(80 + N, N + N // 3 + 2, nchan, fcen, df * nchan, dm)
    got, o, info = _run_both(v, fcen, df * nchan, dm, 4, N, overlap=64, nfront=nfront)
    assert info["fft_len"] == N and info["nfront"] == nfront
    _check(got, o)
    g = cdd.dedisperse(to_dev(np.stack([v, v])), fcen, df * nchan, dm, N, 4, npol=2, overlap=64,
                       nfront=nfront)
    torch.cuda.synchronize()
    assert rel_l2(g["I"].cpu().numpy(), 2 * o["I"]) <= TOL_I


@pytest.mark.parametrize("kind", ["int8", "complex64"])
def test_several_units_taken_at_once(kind):
    """Two beams of many short blocks and two trials each in one persistent launch,
    whose workgroups take several units at a time (also across the beams' border),
    against one call per trial.  Both are FP32 transforms of 256 points, within
    3e-7 of exact intensities each."""
    import torch
    cdd = _cdd()
    fcen, df, dms = 330.0, 0.02, [20.0, 20.5]
    raw = []
    for nchan, nsamp in ((64, 260_001), (48, 250_007)):
        v = torch.from_numpy(np.random.default_rng(nchan).integers(
            -100, 101, size=(nsamp, nchan, 2), dtype=np.int8)).cuda()
        raw.append(torch.view_as_complex(v.float()) if kind == "complex64" else v)
    flush("case: several units at once, %s" % kind)
    plan = cdd.Plan([dict(voltages=v, f_centre=fcen, bw=df * v.shape[1], dms=dms, n_int=2,
                          fft_len=256) for v in raw], single_launch=True)
    plan.execute()
    torch.cuda.synchronize()
    for b, v in enumerate(raw):
        info = plan.info(b)
        for i, dm in enumerate(dms):
            g = cdd.dedisperse(v, fcen, df * v.shape[1], dm, 256, 2, overlap=info["overlap"],
                               nfront=info["nfront"])
            want = g["I"].cpu().numpy()
            assert rel_l2(plan.I[b][i].cpu().numpy()[:want.shape[0]], want) <= 1e-6
    plan.close()
