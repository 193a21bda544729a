"""The long transforms' forms of the chirp and of the detected window, against
the FP64 oracle (tolerances as test_gpu_parity: FP32 transforms of these
lengths stay an order of magnitude below them)."""
import numpy as np
import pytest

import oracle as O
import synth
from tests.test_gpu_parity import TOL_I, TOL_V, _cdd, _check, _run_both
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window", ["none", "welch"])
@pytest.mark.parametrize("blocks", [1, 4, 5])
def test_fullband_chirp_from_the_table_and_in_the_row_pass(blocks, window):
    """Records of up to four blocks form the chirp in the row pass, longer ones
    read the call's table."""
    import torch
    cdd = _cdd()
    nchan, fcen, bw, dm, n_int, N = 128, 610.0, 16.0, 1.0, 16, 1 << 16
    info = cdd.fullband_query(4096, nchan, fcen, bw, dm, n_int, N)
    nspec = (blocks - 1) * info["step"] // (2 * nchan) + 3
    sp = synth.noise_int8(synth.rng_for(6, salt=blocks), nspec, nchan, 20.0)
    flush("case: fullband blocks=%d window=%s" % (blocks, window))
    g = cdd.fullband(to_dev(sp), fcen, bw, dm, n_int, N, taper=window, want_voltages=True)
    torch.cuda.synchronize()
    assert g["info"]["nblocks"] == blocks
    o = O.fullband_dedisperse(sp, fcen, bw, dm, n_int, fft_len=N, overlap=g["info"]["overlap"],
                              nfront=g["info"]["nfront"], window=window, want_voltages=True)
    assert rel_l2(g["y"].cpu().numpy(), o["y"]) <= TOL_V
    assert rel_l2(g["I"].cpu().numpy(), o["P"]) <= TOL_I


@pytest.mark.parametrize("n_int", [1, 2, 4, 8, 16, 32])
@pytest.mark.parametrize("shift", [0, 1, 4, 6])
def test_window_start_against_the_integration_groups(n_int, shift):
    """Window starts on and off the integration groups (split groups, 16-byte
    and single-word sums), a last block cut short, two channels."""
    N, L = 1 << 15, 1024
    rng = np.random.default_rng(10 * n_int + shift)
    v = (rng.standard_normal((2 * (N - L) + 777, 2)) +
         1j * rng.standard_normal((2 * (N - L) + 777, 2))).astype(np.complex64)
    got, o, info = _run_both(v, 610.0, 8.0, 0.05, n_int, N, overlap=L, nfront=512 + shift)
    assert info["nfront"] == 512 + shift
    _check(got, o)


def test_more_items_than_a_launch_takes():
    """Nine blocks of 2^22 points (32 MiB of spectra each) in three channels: two
    launches of each pass, the second from the middle of a channel."""
    N, L, nchan = 1 << 22, 4096, 3
    nsamp = 2 * (N - L) + 777
    v = np.random.default_rng(22).integers(-100, 101, size=(nsamp, nchan, 2), dtype=np.int8)
    got, o, info = _run_both(v, 610.0, 24.0, 0.05, 16, N, want_v=False, overlap=L, nfront=L // 2)
    assert info["nblocks"] == 3
    _check(got, o)
