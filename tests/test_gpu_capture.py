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


def _lists(F, B, seed, n_pool=6):
    """Lists of six kinds; every feature's first one has the most ids."""
    rng = np.random.default_rng(seed)
    pool = [rng.integers(0, 90, n).tolist() for n in (0, 1, 3, 16, 17, 40)]
    rows = [[pool[rng.integers(6)] for _ in range(B)] for _ in range(F)]
    for f in range(F):
        rows[f][0] = pool[5]
    return synth.batch_from_lists(rows)


@pytest.mark.parametrize("kind", ["plain", "runs", "weighted", "grouped"])
@pytest.mark.parametrize("eager_first", [True, False])
def test_captured_builds_outlive_larger_ones(recd, kind, eager_first):
    """A captured build of more than one launch, replayed after eager builds of all kinds with larger tables: it gives what
    an eager build of its batch does.  Also where the capture is the context's first build, which has no tables yet."""
    F, B, group_off, most = 5, 1100, [0, 2, 5], 40 * 5 * 5000
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        c = recd.Context(0, workspace_hint_bytes=recd.workspace_bytes(F, 5000, most, 4))
        c.set_option(recd._OPT_INTERNAL_SMALL_PATH, 0)

    def buffers(batch):
        n, lists = batch.N, batch.F * batch.B
        s = {"values": gu.to_dev(batch.values), "offsets": gu.to_dev(batch.offsets), "weights": torch.ones(n, device="cuda")}
        s["weights"][::7] = 2.0
        s["out"] = [_zeros(n), _zeros(lists + 1), _zeros(lists, torch.int32), _zeros(batch.F + 1)]
        s["u_weights"], s["runs"] = _zeros(n, torch.float32), _zeros(3 * (lists + 2))
        s["inverse_g"], s["group_uoff"] = _zeros(2 * batch.B, torch.int32), _zeros(3)
        return s

    def build(kind, s, B):
        uv, uo, inv, fu = s["out"]
        if kind == "plain":
            c.build_ikjt(F, B, s["values"], s["offsets"], *s["out"])
        elif kind == "runs":
            c.build_ikjt_runs(F, B, s["values"], s["offsets"], *s["out"], s["runs"])
        elif kind == "weighted":
            c.build_ikjt_weighted(F, B, s["values"], s["weights"], s["offsets"], uv, s["u_weights"], uo, inv, fu)
        else:
            c.build_ikjt_grouped(F, B, group_off, s["values"], s["offsets"], uv, uo, s["inverse_g"], s["group_uoff"], fu, inv)

    def results(s):
        torch.cuda.synchronize()
        out = [*s["out"], s["u_weights"], s["runs"], s["inverse_g"], s["group_uoff"]]
        got = [x.clone() for x in out]
        for x in out:
            x.zero_()
        return got

    try:
        with torch.cuda.stream(stream):
            batches = [_lists(F, B, 0)]
            s = buffers(batches[0])
            if kind == "grouped":   # its groups are on the device before a capture
                tiny = _lists(F, 3, 9)
                build(kind, buffers(tiny), 3)
            if eager_first:
                build(kind, s, B)
                results(s)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                build(kind, s, B)
            for seed in range(1, 5):
                if seed > 1:
                    big = _lists(F, 1200 * seed, seed)
                    b = buffers(big)
                    for k in ("plain", "weighted", "grouped"):
                        build(k, b, big.B)
                    torch.cuda.synchronize()
                lists = batches[0].offsets[1:] - batches[0].offsets[:-1]
                s["values"].copy_(torch.from_numpy(np.random.default_rng(seed).integers(0, 3, batches[0].N)))
                if seed % 2:
                    s["offsets"][1:].copy_(torch.cumsum(torch.from_numpy(lists[::-1].copy()).cuda(), 0))
                graph.replay()
                got = results(s)
                graph.replay()
                again = results(s)
                build(kind, s, B)
                want = results(s)
                assert int(want[3][-1]) > F
                assert all(torch.equal(x, y) for x, y in zip(got, want)) and all(torch.equal(x, y) for x, y in zip(again, want))
    finally:
        c.close()
