"""The queue entries of a state snapshot as the binding hands them out: every
field of the packed entries, over their whole ranges (a library stand-in fills
the buffers; no GPU)."""
import ctypes

import numpy as np
import pytest

from paper_2606_11440_amd import _lib


@pytest.mark.parametrize("E,M,qcap", [(0, 3, 4), (1, 1, 1), (2, 3, 5), (7, 5, 64)])
def test_queue_fields(monkeypatch, E, M, qcap):
    r = np.random.default_rng(E + qcap)
    want = np.zeros(E * M * qcap, _lib.ENTRY_DT)
    for f in ("key", "id", "t_arr"):
        want[f] = r.integers(-2 ** 31, 2 ** 31, want.size)
    want["svc"] = r.integers(0, 2 ** 16, want.size)
    want["budget"] = r.integers(-2 ** 15, 2 ** 15, want.size)
    if want.size > 3:
        want["svc"][:4], want["budget"][:4] = (0, 65535, 1, 65535), (-32768, -1, 32767, 0)

    class Library:
        @staticmethod
        def im_read_state(pool, begin, count, tick, envs, models, slots, queues, hist):
            ctypes.memmove(queues, want.ctypes.data, want.nbytes)
            return 0

    monkeypatch.setattr(_lib, "load", lambda: Library)
    q = _lib.im_read_state(None, 0, E, M, 2 * M, 3, qcap, M)["queues"]
    assert q.shape == (E, M, qcap, 5) and q.dtype == np.int32 and q.flags.c_contiguous
    for i, f in enumerate(("key", "id", "t_arr", "svc", "budget")):
        np.testing.assert_array_equal(q[..., i].reshape(-1), want[f].astype(np.int32))
