"""A block counts as queued work from the moment a push takes its slot: callers
that wait for queued work, or end the server, while another thread's push is
still copying its block wait for that block.  The results are those of the
whole-record call (the two chirp forms differ by FP32 rounding: 1e-6 relative
L2)."""
import threading
import time

import numpy as np
import pytest

from tests.test_gpu_parity import _cdd
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu
NCHAN, FCEN, BW, DM, N_INT = 512, 325.0, 32.0, 5.0, 4


def _push_under_way(cdd, nsamp):
    """A server, its one stream and a thread some milliseconds before the end of
    the push of one large block (512 MB: 12 ms of copying and more)."""
    x = np.random.default_rng(3).integers(-60, 61, size=(nsamp, NCHAN, 2), dtype=np.int8)
    sv = cdd.Server(queue_depth=1)
    sid = sv.open(cdd.CDD_CI8, NCHAN, FCEN, BW, DM, N_INT, nsamp)
    begun, res = threading.Event(), []

    def push():
        begun.set()
        try:
            res.append(sv.push(sid, x, 0))
        except cdd.CddError as e:
            res.append(e)

    th = threading.Thread(target=push)
    th.start()
    begun.wait()
    time.sleep(0.002)
    return sv, sid, th, res, x


def test_close_and_sync_wait_for_a_block_being_copied():
    import torch
    cdd = _cdd()
    flush("case: close and sync during a push")
    sv, sid, th, res, x = _push_under_way(cdd, 1 << 19)
    sv.close_stream(sid)
    sv.sync()
    got = sv.poll(sid)[1]
    th.join(60)
    assert not th.is_alive() and res == [0], res
    sv.close()
    o = cdd.dedisperse(to_dev(x), FCEN, BW, DM, 0, N_INT)
    torch.cuda.synchronize()
    want = o["I"].cpu().numpy().astype(np.float64)
    assert got.shape == want.shape
    assert rel_l2(got, want) <= 1e-6


def test_destroy_waits_for_a_block_being_copied():
    cdd = _cdd()
    flush("case: destroy during a push")
    sv, _, th, res, _ = _push_under_way(cdd, 1 << 19)
    sv.close()
    th.join(60)
    assert not th.is_alive() and res == [0], res
