"""Builders and stream capture: calls beside a capture, and captured builds that are replayed after larger ones."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2211_05239_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def recd():
    from paper_2211_05239_amd import recd as mod
    return mod


def _zeros(n, dt=torch.int64):
    return torch.zeros(n, dtype=dt, device="cuda")


def test_builds_on_the_null_stream_beside_a_capture(recd):
    """While another stream is being captured a context on the null stream builds as ever."""
    hip = recd._lib  # the runtime that the library is linked against
    stream, graph = C.c_void_p(), C.c_void_p()
    F, B = 2, 4
    batch = synth.batch_from_lists([[[1, 2], [1, 2], [3], []], [[5], [5], [5], []]])
    values, offsets = gu.to_dev(batch.values), gu.to_dev(batch.offsets)
    grouped = [_zeros(batch.N), _zeros(F * B + 1), _zeros(B, torch.int32), _zeros(2), _zeros(F + 1)]
    plain = [_zeros(batch.N), _zeros(F * B + 1), _zeros(F * B, torch.int32), _zeros(F + 1)]
    c = recd.Context(0, stream=0)
    c.set_option(recd._OPT_INTERNAL_SMALL_PATH, 0)

    def build():
        c.build_ikjt_grouped(F, B, [0, 2], values, offsets, *grouped)
        c.build_ikjt(F, B, values, offsets, *plain)
    try:
        build()
        torch.cuda.synchronize()
        want = [x.clone() for x in grouped + plain]
        assert want[2].tolist() == [0, 0, 1, 2]
        for x in grouped + plain:
            x.zero_()
        torch.cuda.synchronize()
        assert hip.hipStreamCreate(C.byref(stream)) == 0
        assert hip.hipStreamBeginCapture(stream, 2) == 0  # relaxed
        try:
            build()
        finally:
            assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
            hip.hipGraphDestroy(graph)
            hip.hipStreamDestroy(stream)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(grouped + plain, want))
    finally:
        c.close()
