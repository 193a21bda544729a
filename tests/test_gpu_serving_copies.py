"""Pushes large enough to be copied by several threads and in two halves, from
two callers at once, against the whole-record call (the same kernels on the
same samples; the two chirp forms differ by FP32 rounding: 1e-6 relative L2)."""
import threading

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import _cdd
from tests.util import flush, rel_l2, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [8193, 2731, 1023])
def test_large_pushes_from_two_threads(block):
    import torch
    cdd = _cdd()
    nchan, fcen, bw, dm, n_int, blocks = 512, 325.0, 32.0, 5.0, 4, 5
    recs = [synth.noise_int8(synth.rng_for(5, salt=block + k), block * blocks - 7 * k, nchan, 20.0)
            for k in range(2)]
    flush("case: two threads pushing blocks of %d samples" % block)
    sv = cdd.Server()
    got, errs = [None, None], []

    def feed(k):
        try:
            sid = sv.open(cdd.CDD_CI8, nchan, fcen, bw, dm, n_int, block)
            parts = []
            for b in range(blocks):
                while sv.push(sid, recs[k][b * block:(b + 1) * block], b) != 0:
                    parts.append(sv.poll(sid)[1])
            sv.close_stream(sid)
            total = len(recs[k]) // n_int
            while sum(len(p) for p in parts) < total:
                sv.sync()
                parts.append(sv.poll(sid)[1])
            got[k] = np.concatenate(parts)
        except Exception as e:  # noqa: BLE001
            errs.append(e)

    th = [threading.Thread(target=feed, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join(60)
    assert not errs and all(not t.is_alive() for t in th), errs
    sv.close()
    for k in range(2):
        o = cdd.dedisperse(to_dev(recs[k]), fcen, bw, dm, 0, n_int)
        torch.cuda.synchronize()
        assert rel_l2(got[k], o["I"].cpu().numpy().astype(np.float64)) <= 1e-6
